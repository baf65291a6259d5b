"""Builds libsage.so (the C-ABI library of hand-written gfx950 kernels) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsage.so")
SOURCES = ["sage_api.hip", "sage_prepass.hip", "sage_prepass_v.hip", "sage_attn.hip", "sage_attn_pv8.hip",
           "sage_decode.hip", "sage_short.hip", "sage_microbench.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off",                                   # quantizer arithmetic: one rounding per operation
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 code generation
    "-mllvm", "-amdgpu-mfma-vgpr-form",                    # scores must land in VALU-readable registers
    "-Wall", "-Wno-unused-variable",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


HASH_MARKER = b"SAGE_SOURCE_HASH="


def source_files() -> list:
    """Everything the library is compiled from: the kernel sources and headers, and the public header."""
    names = sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".h")))
    return [os.path.join(CSRC, f) for f in names] + [os.path.join(HERE, "..", "include", "sage.h")]


def source_hash() -> str:
    """SHA-256 over the names and contents of source_files(); compiled into the library, so that a
    built library can be matched against the sources beside it whatever the file times say."""
    import hashlib
    h = hashlib.sha256()
    for path in source_files():
        h.update(os.path.basename(path).encode() + b"\0")
        with open(path, "rb") as f:
            h.update(f.read())
        h.update(b"\0")
    return h.hexdigest()


def built_hash(path: str = LIB, marker: bytes = HASH_MARKER):
    """The source hash a built library carries (read from the file, nothing is loaded), or None."""
    if not os.path.exists(path):
        return None
    with open(path, "rb") as f:
        blob = f.read()
    at = blob.find(marker)
    if at < 0:
        return None
    digest = blob[at + len(marker): at + len(marker) + 64]
    try:
        return digest.decode("ascii")
    except UnicodeDecodeError:
        return None


NATIVE = os.path.join(HERE, "_sage_native.so")
NATIVE_SOURCE = os.path.join(CSRC, "binding.cpp")
NATIVE_MARKER = b"SAGE_NATIVE_HASH="


def native_hash() -> str:
    """SHA-256 over what the extension module is compiled from and against: its source, the public header, and
    the versions of torch and Python."""
    import hashlib
    import torch
    h = hashlib.sha256(f"{torch.__version__} {sys.version}".encode())
    for path in (NATIVE_SOURCE, os.path.join(HERE, "..", "include", "sage.h")):
        with open(path, "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def native_is_stale() -> bool:
    return built_hash(NATIVE, NATIVE_MARKER) != native_hash()


def build_native() -> str:
    """Compile the Python extension module (host code only) and return its path."""
    import sysconfig
    import torch
    root = os.path.dirname(torch.__file__)
    tmp = NATIVE + ".tmp.%d" % os.getpid()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", f'-DSAGE_NATIVE_HASH="{native_hash()}"',
           "-I" + os.path.join(root, "include"), "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-I" + sysconfig.get_paths()["include"], "-o", tmp, NATIVE_SOURCE,
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"]
    try:
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("g++ failed:\n" + res.stderr)
        os.replace(tmp, NATIVE)
    finally:
        if os.path.exists(tmp):
            os.remove(tmp)
    return NATIVE


def build(verbose: bool = False, extra=()) -> str:
    """Compile every kernel for gfx950 (cross-compiles without a GPU), then the extension module, and return the
    library's path."""
    build_library(verbose, extra)
    build_native()
    return LIB


def build_library(verbose: bool = False, extra=()) -> str:
    """Compile every kernel and return the library's path."""
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [hipcc(), *HIPCC_FLAGS, *extra, f'-DSAGE_SOURCE_HASH="{source_hash()}"', "-o", tmp,
           *[os.path.join(CSRC, s) for s in SOURCES]]
    try:
        res = subprocess.run(cmd, capture_output=True, text=True)
        noise = "packed-fp32-ops"
        err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + err)
        if verbose and err.strip():
            print(err, file=sys.stderr)
        verify_attention_isa(extra)
        os.replace(tmp, LIB)
    finally:
        if os.path.exists(tmp):         # a failed build or a failed assembly check leaves nothing behind
            os.remove(tmp)
    return LIB


# The attention kernels that are built: the score dump for head dimension {64, 128} x {4, 8 wavefronts}; {causal, full} x
# {per-block, per-token key scales} for D = 64 with 4 wavefronts and D = 128 with 4 and 8; the two measurement builds (D =
# 128, 8 wavefronts, causal / full, with the clock counters).  Beside them TWO_SET_KERNELS: {causal, full} x {per-block,
# per-token} for D = 64 with two sets of 4 wavefronts, known by their last template argument.
ATTENTION_KERNELS = 4 + 4 * 3 + 2
TWO_SET_KERNELS = 4
TWO_SETS = "ELb0ELi2EEEv"


def _registers(operand: str, file: str) -> set:
    """Numbers of the registers of a file ("v" or "a") that an operand such as v12 or a[12:15] names."""
    import re
    m = re.fullmatch(file + r"(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return set()
    return {int(m.group(1))} if m.group(1) else set(range(int(m.group(2)), int(m.group(3)) + 1))


def _operands(code: str) -> list:
    parts = code.split(None, 1)
    return [o.strip() for o in parts[1].split(",")] if len(parts) > 1 else []


class MatrixHazards:
    """The waits that the compiler would insert if it knew that inline assembly holds matrix instructions, checked over a
    kernel's instructions in the order of the text:
      - no instruction touches a VGPR within 12 wait states of a matrix instruction writing it (except the next matrix
        instruction of the same accumulation chain), where either of the two is the source's own,
      - none of the source's own matrix instructions reads a VGPR that one of the two preceding instructions wrote.
    Between instructions that it placed itself the compiler sees to the waits."""

    def __init__(self, kernel: str, problems: list):
        self.kernel, self.problems = kernel, problems
        self.pending = []         # [registers written by a matrix instruction, wait states since, its text, source's own]
        self.recent = []          # VGPRs written by the last two non-matrix instructions

    def branch(self, code: str) -> None:
        """A label ("") or a branch."""
        if code.startswith("s_branch"):
            self.pending, self.recent = [], []          # nothing falls through an unconditional branch
        elif code:
            for p in self.pending:
                p[1] += 1

    def instruction(self, code: str, own: bool) -> None:
        """own: a matrix instruction that the source wrote."""
        import re
        ops = _operands(code)
        touched = set().union(*[_registers(o, "v") for o in ops]) if ops else set()
        is_mfma = code.startswith("v_mfma")
        own = own and is_mfma
        for written, waited, text, theirs in self.pending:
            same_chain = is_mfma and _registers(ops[0], "v") == written and _registers(ops[-1], "v") == written
            if touched & written and not same_chain and (own or theirs):
                self.problems.append(f"{self.kernel}: '{code}' touches the result of '{text}' after {waited} wait states")
        if own and any(_registers(o, "v") & w for o in ops[1:] for w in self.recent):
            self.problems.append(f"{self.kernel}: '{code}' reads a register written less than 2 wait states before")
        m = re.match(r"s_nop\s+(\d+)", code)
        step = int(m.group(1)) + 1 if m else 1
        for p in self.pending:
            p[1] += step
        dst = _registers(ops[0], "v") if is_mfma else set()
        # (a result that the chain's next instruction has taken over is that one's)
        self.pending = [p for p in self.pending if p[1] < 12 and p[0] != dst]
        if is_mfma:
            if dst:
                self.pending.append([dst, 0, code, own])
            self.recent = []
        else:
            wrote = _registers(ops[0], "v") if ops and code.startswith("v_") else set()      # VALU results only: loads are covered by s_waitcnt
            self.recent = ([wrote] + self.recent)[:2] if step == 1 else []


def check_attention_asm(text: str) -> list:
    """Checks the assembly text of the attention kernels for what their hand-placed register use
    relies on (see "Register files" at the top of sage_attn.hip) and returns the list of problems
    found.  The matrix instructions update accumulator registers that they name as inputs, so the
    compiler must keep every accumulator in one place between them:
      - once the first matrix instruction has been issued it never copies an accumulator register
        to another accumulator register (before that, the zero initialisation may),
      - it reads accumulator registers into VGPRs only where the source refreshes them first (the
        rare rescale and the epilogue), i.e. never inside a block that issues matrix instructions
        (AGPRs that no matrix instruction names are the compiler's own parking space and exempt),
      - nothing spills to scratch memory,
      - it never touches m0, which the hand-written global->LDS loads set,
      - and the waits are there that the compiler does not know of (MatrixHazards).
    Instructions between ";;#ASMSTART" and ";;#ASMEND" are the source's own assembly."""
    import re
    kernels = re.findall(r"^(_ZN4sage16sage_attn_kernel\w+):.*?^\.Lfunc_end\d+:", text, re.S | re.M)
    bodies = re.findall(r"^_ZN4sage16sage_attn_kernel\w+:.*?^\.Lfunc_end\d+:", text, re.S | re.M)
    problems = []
    one_set = sum(TWO_SETS not in name for name in kernels)
    if one_set != ATTENTION_KERNELS:
        problems.append(f"expected {ATTENTION_KERNELS} attention kernels in the assembly, found {one_set}")

    for name, body in zip(kernels, bodies):
        # AGPRs that matrix instructions name (accumulators, resident operands).  The compiler may
        # park unrelated values in the remaining AGPRs; moving those around is harmless.
        matrix_agprs = set()
        for line in body.split("\n"):
            code = line.split(";")[0].strip()
            if code.startswith("v_mfma"):
                for o in _operands(code):
                    matrix_agprs |= _registers(o, "a")
        state = {"mfma": False, "reads": []}
        in_asm = False
        seen_mfma = False
        hazards = MatrixHazards(name, problems)

        def close_block():
            if state["mfma"] and state["reads"]:
                problems.append(f"{name}: accumulator read next to matrix instructions: {state['reads'][0]}")
            state["mfma"], state["reads"] = False, []

        for line in body.split("\n"):
            code = line.split(";")[0].strip()
            if "#ASMSTART" in line:
                in_asm = True
                continue
            if "#ASMEND" in line:
                in_asm = False
                continue
            if re.match(r"^\.LBB\d+_\d+:", line) or code.startswith("s_cbranch") or code.startswith("s_branch"):
                close_block()
                hazards.branch("" if code.startswith(".") else code)
                continue
            if not code or code.startswith("."):
                continue
            hazards.instruction(code, True)
            is_mfma, ops = code.startswith("v_mfma"), _operands(code)
            # --- register-file rules
            if in_asm:
                if is_mfma:
                    state["mfma"] = True
                    seen_mfma = True
                continue
            named = set().union(*[_registers(o, "a") for o in ops]) if ops else set()
            if code.startswith("v_accvgpr_mov") and seen_mfma and named & matrix_agprs:
                problems.append(f"{name}: accumulator-to-accumulator copy: {code}")
            if code.startswith("v_accvgpr_read") and named & matrix_agprs:
                state["reads"].append(code)
            if code.startswith("scratch_"):
                problems.append(f"{name}: scratch access: {code}")
            if re.search(r"\bm0\b", code):
                problems.append(f"{name}: compiler-generated use of m0: {code}")
        close_block()
    return problems


# Registers (VGPRs and AGPRs together) with which three workgroups of 4 wavefronts fit on a CU: 512 / 3, in steps of 8.
THREE_WORKGROUPS_VGPRS = 168


def check_attention_registers(text: str) -> list:
    """The attention kernels of D = 64 run three workgroups on a CU; their launch bounds ask for two, so nothing but this keeps
    the compiler within the registers of three."""
    import re
    used = re.findall(r"^\s*\.amdhsa_kernel (_ZN4sage16sage_attn_kernelILi64ELi4ELb[01]ELb0E\w+).*?^\s*\.amdhsa_next_free_vgpr (\d+)", text, re.S | re.M)
    problems = [f"{name}: {n} registers, with which two workgroups fit on a CU instead of three" for name, n in used
                if int(n) > THREE_WORKGROUPS_VGPRS]
    if len(used) != 4:
        problems.append(f"expected the register counts of 4 attention kernels with D = 64, found {len(used)}")
    return problems


def check_two_sets(text: str) -> list:
    """All attention kernels with two sets of wavefronts are in the text that check_attention_asm() looks through."""
    import re
    found = sum(TWO_SETS in name for name in re.findall(r"^(_ZN4sage16sage_attn_kernel\w+):", text, re.M))
    return [] if found == TWO_SET_KERNELS else [f"expected {TWO_SET_KERNELS} attention kernels with two sets of wavefronts, found {found}"]


def check_loads_asm(text: str, kernel: str, expected: int) -> list:
    """Checks the assembly text of `kernel`'s instantiations, whose matrix instructions are compiler builtins but for the
    seeded ones of the INT8 second product: that nothing spills to scratch memory, that the compiler never touches m0, which
    the hand-written global->LDS loads set, and that the waits around hand-written matrix instructions are there."""
    import re
    bodies = re.findall(rf"^(_ZN4sage{len(kernel)}{kernel}\w+):(.*?)^\.Lfunc_end\d+:", text, re.S | re.M)
    problems = []
    if len(bodies) != expected:
        problems.append(f"expected {expected} instantiations of {kernel} in the assembly, found {len(bodies)}")
    for name, body in bodies:
        in_asm = False
        hazards = MatrixHazards(name, problems)
        for line in body.split("\n"):
            if "#ASMSTART" in line:
                in_asm = True
                continue
            if "#ASMEND" in line:
                in_asm = False
                continue
            code = line.split(";")[0].strip()
            if re.match(r"^\.LBB\d+_\d+:", line) or code.startswith("s_cbranch") or code.startswith("s_branch"):
                hazards.branch("" if code.startswith(".") else code)
                continue
            if not code or code.startswith("."):
                continue
            hazards.instruction(code, in_asm)
            if in_asm:
                continue
            if code.startswith("scratch_"):
                problems.append(f"{name}: scratch access: {code}")
            if re.search(r"\bm0\b", code):
                problems.append(f"{name}: compiler-generated use of m0: {code}")
    return problems


def check_pv8_asm(text: str) -> list:
    """The INT8-P~V attention kernels: head dimension {64, 128} x {causal, full} x {per-block, per-token key scales} x {whole,
    key chunks}."""
    return check_loads_asm(text, "sage_attn_pv8_kernel", 16)


def check_short_asm(text: str) -> list:
    """The whole-pass kernels for short sequences: {128, 256, 512 keys at D = 64, 128, 256 at D = 128} x {per-block, per-token
    key scales}."""
    return check_loads_asm(text, "sage_short_kernel", 10)


def check_short_pair_asm(text: str) -> list:
    """The same with two wavefronts per query tile: {256, 512 keys at D = 64} x {per-block, per-token key scales}."""
    return check_loads_asm(text, "sage_short_pair_kernel", 4)


def check_decode_asm(text: str) -> list:
    """The kernels for few queries: {4 wavefronts at D = 64, 2 and 4 at D = 128} x {per-block, per-token key scales}; and the
    merge of key chunks beside them, which has no loads of that kind."""
    return check_loads_asm(text, "sage_decode_kernel", 6) + check_no_spills(text)


def check_no_spills(text: str) -> list:
    """The pre-pass kernels hold a quantization block in registers; a register spill would turn the
    one pass over memory they are built around into several.  Returns the kernels that touch scratch."""
    import re
    problems = []
    for m in re.finditer(r"^(_ZN4sage\w+):.*?^\.Lfunc_end\d+:", text, re.S | re.M):
        if "scratch_" in m.group(0):
            problems.append(f"{m.group(1)}: scratch access (register spill)")
    return problems


def verify_attention_isa(extra=()) -> None:
    """Compiles the kernel sources to assembly and raises RuntimeError if check_attention_asm(),
    check_loads_asm() or check_no_spills() objects."""
    import tempfile
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    problems = []
    with tempfile.TemporaryDirectory() as tmp:
        for src, check in (("sage_attn.hip", lambda s: check_attention_asm(s) + check_attention_registers(s) + check_two_sets(s)), ("sage_attn_pv8.hip", check_pv8_asm),
                           ("sage_prepass.hip", check_no_spills), ("sage_prepass_v.hip", check_no_spills),
                           ("sage_short.hip", check_short_asm), ("sage_short.hip", check_short_pair_asm), ("sage_decode.hip", check_decode_asm)):
            out = os.path.join(tmp, src + ".s")
            cmd = [hipcc(), *flags, *extra, "-S", "--cuda-device-only", "-o", out, os.path.join(CSRC, src)]
            res = subprocess.run(cmd, capture_output=True, text=True)
            if res.returncode != 0:
                raise RuntimeError("hipcc -S failed:\n" + res.stderr)
            problems += check(open(out).read())
    if problems:
        raise RuntimeError("attention kernel ISA check failed:\n  " + "\n  ".join(problems[:20]))


def is_stale() -> bool:
    """True when there is no built library or it was not built from the sources as they are now."""
    return built_hash() != source_hash()


def have_compiler() -> bool:
    import shutil
    cc = hipcc()
    return os.path.exists(cc) if os.path.isabs(cc) else shutil.which(cc) is not None


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
