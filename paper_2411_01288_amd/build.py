"""Builds libhexa_moe.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import re
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhexa_moe.so")
SOURCES = ["api.hip", "index.hip", "elementwise.hip", "f32_path.hip", "gemm_bf16.hip", "probe.hip", "route.hip",
           "bench_support.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


# The contraction kernels count their own direct-to-LDS loads in vmcnt; a register spill inside
# their K loop would add vector-memory operations the count does not know about.  So the build
# refuses a gemm_bf16.hip whose kernels use any scratch memory at all.  It also refuses scalar
# register spills: a spilled scalar comes back through v_readlane, and a vector-memory instruction
# must not read a scalar register within five wait states of a vector instruction writing it; the
# compiler pads that hazard in front of its own loads, but the staging loads are inline assembly
# (a reloaded resource word or offset read too early fetched the previous tile's rows).  (About 1 KB of scratch per
# lane in one instantiation means its K loop was left rolled: LLVM ignores "#pragma unroll" past a
# size threshold, -mllvm -pragma-unroll-threshold=N, and the accumulator and fragment arrays are
# then indexed dynamically and live in scratch.)  The fp32 path's 128x64 tiles keep sums in inline assembly's
# registers (see lint_asm_mfma), with few to spare: a spill would stand between those instructions.
NO_SCRATCH = {"gemm_bf16.hip": "gemm_bf16", "f32_path.hip": "f32_gemm"}   # source: its kernels' common name


def _compile(src: str) -> str:
    obj = os.path.join(CSRC, src.replace(".hip", ".o"))
    cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    if src not in NO_SCRATCH:
        subprocess.check_call(cmd)
        return obj
    res = subprocess.run(cmd + ["-Rpass-analysis=kernel-resource-usage"], stderr=subprocess.PIPE, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{res.stderr}")
    name, bad = None, []
    for line in res.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"(ScratchSize \[bytes/lane\]|SGPRs Spill|VGPRs Spill): (\d+)", line)
        if m and int(m.group(2)) > 0 and name and NO_SCRATCH[src] in name:
            bad.append((name, m.group(1), int(m.group(2))))
    if bad:
        raise RuntimeError(f"{src}: kernels spill registers: {bad}")
    return obj


def _sgprs(text: str):
    """Scalar register numbers named in an operand string: s7, s[4:7]."""
    regs = set()
    for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        regs.update(range(int(a), int(b) + 1))
    regs.update(int(n) for n in re.findall(r"\bs(\d+)\b", text))
    return regs


def _vgprs(text: str):
    """Vector register numbers named in an operand string: v7, v[4:7]."""
    regs = set()
    for a, b in re.findall(r"\bv\[(\d+):(\d+)\]", text):
        regs.update(range(int(a), int(b) + 1))
    regs.update(int(n) for n in re.findall(r"\bv(\d+)\b", text))
    return regs


def lint_asm_hazards(text: str) -> list:
    """Wait-state hazards in generated ISA that the compiler's hazard recogniser does not cover, as a list of
    (line, instruction, registers); empty when there is none.

    1. A vector-memory instruction must not read a scalar register within five wait states of a VECTOR
       instruction writing it (v_readfirstlane of a uniform value kept in vector registers, v_readlane of a
       spilled scalar).  Checked for the inline-assembly loads and stores: the direct-to-LDS staging
       loads, global loads with a scalar base (the row-offset loads), buffer stores.
    2. A vector instruction must not write a data register of a store of more than 8 bytes within two wait
       states behind it.  (The compiler leaves no gap where a buffer store's scalar offset is a register.)"""
    window = []   # (wait states this instruction provides, scalar registers a vector instruction wrote)
    stores = []   # (wait states since the store, its data registers, text)
    bad = []
    for ln, line in enumerate(text.splitlines(), 1):
        t = line.strip()
        if not t or t[0] in ";." or t.endswith(":") or t.startswith(("//", "#")):
            if t.endswith(":"):
                window = []          # a label: the predecessors are unknown, start over
            continue
        op = t.split()[0]
        ops = t.split(None, 1)[1] if " " in t or "\t" in t else ""
        if ((op.startswith("buffer_load") and t.endswith("lds")) or (op.startswith("global_load") and "s[" in t)
                or op.startswith("buffer_store")):
            need, used = 5, _sgprs(ops)
            for states, written in reversed(window):
                if need <= 0:
                    break
                if written & used:
                    bad.append((ln, t, sorted(written & used)))
                    break
                need -= states
        written = set()
        if op.startswith(("v_readfirstlane", "v_readlane")) or (op.startswith("v_cmp") and "_e64" in op):
            written = _sgprs(ops.split(",")[0])
        elif op.startswith("v_"):
            vec = _vgprs(ops.split(",")[0])
            bad += [(ln, f"{txt} | {t}", sorted(vec & data)) for states, data, txt in stores if vec & data]
        states = 1
        if op == "s_nop":
            states = int(t.split()[1]) + 1
        window.append((states, written))
        del window[:-8]
        stores = [(n + states, data, txt) for n, data, txt in stores if n + states < 2]
        if re.match(r"(buffer|global|flat)_store_dwordx[34]", op):
            stores.append((0, _vgprs(ops.split(",")[0 if op.startswith("buffer") else 1]), t))
    return bad


# v_mfma_f32_16x16x32_bf16 (8 passes) on gfx950: wait states from it to any other instruction that reads or writes its result, to a matrix
# instruction that adds to exactly it, and from a vector instruction that writes one of its operands to it.
MFMA_RESULT, MFMA_CHAIN, MFMA_OPERAND = 12, 2, 2


def lint_asm_mfma(text: str) -> list:
    """Wait states around matrix instructions written as inline assembly (between the compiler's ASMSTART and ASMEND), which its hazard
    recogniser takes for any instruction: (line, matrix instruction, the other one, registers) of every violation, along all paths."""
    ops, labels, asm = [], {}, False
    for ln, line in enumerate(text.splitlines(), 1):
        t = line.strip()
        if t.startswith(";;#ASM"):
            asm = t.startswith(";;#ASMSTART")
            continue
        t = t.split(";")[0].split("//")[0].strip()
        if t.endswith(":"):
            labels[t[:-1]] = len(ops)
        elif t and t[0] not in ".#":
            ops.append((ln, t, asm))
    names = [t.split()[0] for _, t, _ in ops]
    after = [[] if n in ("s_branch", "s_endpgm", "s_setpc_b64") else [i + 1] for i, n in enumerate(names)]
    before = [[] for _ in range(len(ops) + 1)]
    for i, n in enumerate(names):
        if n.startswith(("s_cbranch", "s_branch")):
            after[i].append(labels[ops[i][1].split()[1]])
        for j in after[i]:
            before[j].append(i)
    states = [int(t.split()[1], 0) + 1 if n == "s_nop" else 1 for n, (_, t, _) in zip(names, ops)]
    regs = [[_vgprs(o) for o in t.split(None, 1)[1].split(",")] if n.startswith(("v_", "ds_", "buffer_", "global_", "flat_", "scratch_")) else []
            for n, (_, t, _) in zip(names, ops)]
    bad = []

    def walk(first, edges, most, visit):
        seen, todo = {}, [(j, 0) for j in first]
        while todo:
            j, gone = todo.pop()
            if gone >= most or j >= len(ops) or seen.get(j, most) <= gone:
                continue
            seen[j] = gone
            visit(j, gone)
            todo += [(n, gone + states[j]) for n in edges[j]]

    for i, (ln, t, asm) in enumerate(ops):
        if not (asm and names[i].startswith("v_mfma")):
            continue
        result, operands = regs[i][0], set().union(*regs[i][1:])

        def reader(j, gone):
            used = set().union(*regs[j])
            chain = names[j].startswith("v_mfma") and regs[j][3] == result and not result & (regs[j][1] | regs[j][2])
            if gone < (MFMA_CHAIN if chain else MFMA_RESULT) and used & result:
                bad.append((ln, t, ops[j][1], sorted(used & result)))

        def writer(j, gone):
            if names[j].startswith("v_") and not names[j].startswith("v_mfma") and regs[j][0] & operands:
                bad.append((ln, t, ops[j][1], sorted(regs[j][0] & operands)))

        walk(after[i], after, MFMA_RESULT, reader)
        walk(before[i], before, MFMA_OPERAND, writer)
    return bad


def lint_staging_hazards(src: str) -> None:
    """Refuses the build if the generated ISA of `src` holds a hazard (see lint_asm_hazards, lint_asm_mfma)."""
    res = subprocess.run(["hipcc", *FLAGS, "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", "-"],
                         stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc -S failed on {src}")
    bad = lint_asm_hazards(res.stdout) + lint_asm_mfma(res.stdout)
    if bad:
        raise RuntimeError(f"{src}: wait-state hazards: {bad[:5]}")


MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))   # (another Python does not look for it)


def build_marshal() -> str:
    """_marshal.*.so: the argument marshalling of binding.py (host code, against the installed torch, whose version it keeps)."""
    import torch
    from torch.utils.cpp_extension import include_paths
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-fPIC", "-shared", "-fvisibility=hidden",
                           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                           f'-DBUILT_FOR_TORCH="{torch.__version__}"',
                           *(f"-isystem{d}" for d in [*include_paths(), sysconfig.get_paths()["include"]]),
                           os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL,
                           f"-L{lib}", f"-Wl,-rpath,{lib}", "-ltorch_python", "-ltorch_cpu", "-lc10"])
    return MARSHAL


def build_library(jobs: int = 8) -> str:
    """Compile every translation unit and link the shared library and the binding's marshalling.  Always rebuilds."""
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        lints = [ex.submit(lint_staging_hazards, src) for src in NO_SCRATCH]
        marshal = ex.submit(build_marshal)
        objs = list(ex.map(_compile, SOURCES))
        for lint in lints:
            lint.result()
        marshal.result()
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


# ---- host-code sanitizer build (CPU-side checks only; the device code is compiled as usual) ----
SAN_LIB = os.path.join(HERE, "libhexa_moe_asan.so")
SAN_HOST = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
            "-Xarch_host", "-fno-sanitize-recover=undefined"]


def sanitizer_runtime() -> str:
    """Path of the AddressSanitizer runtime that the sanitized library needs preloaded."""
    out = subprocess.check_output(["/opt/rocm/llvm/bin/clang++", "-print-file-name=libclang_rt.asan-x86_64.so"],
                                  text=True).strip()
    if not os.path.exists(out):
        raise RuntimeError("clang's AddressSanitizer runtime was not found")
    return out


def build_sanitized_library(jobs: int = 7) -> str:
    """libhexa_moe_asan.so: the same sources with AddressSanitizer and UndefinedBehaviorSanitizer on the
    host code (argument checks, workspace layout, launch set-up), and the binding's marshalling (as always).
    tests/test_sanitizers.py runs the host-only ABI tests against it; GPU sanitizers are not used."""
    def one(src: str) -> str:
        obj = os.path.join(CSRC, src.replace(".hip", ".asan.o"))
        flags = [f for f in FLAGS if f != "-O3"] + ["-O1", "-g", "-fno-omit-frame-pointer"]
        subprocess.check_call(["hipcc", *flags, *SAN_HOST, "-c", os.path.join(CSRC, src), "-o", obj])
        return obj
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        marshal = ex.submit(build_marshal)
        objs = list(ex.map(one, SOURCES))
        marshal.result()
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-fsanitize=address,undefined", "-fno-gpu-sanitize",
                           "-shared-libsan", "-o", SAN_LIB, *objs])
    return SAN_LIB


if __name__ == "__main__":
    import sys
    print(build_sanitized_library() if "--sanitize" in sys.argv[1:] else build_library())
