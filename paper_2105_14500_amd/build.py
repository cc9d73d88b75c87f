"""Compile the HIP library for gfx950 into paper_2105_14500_amd/libtesseract_hip.so, and the native
argument marshalling of the Python binding beside it (_tess_call.so)."""
import concurrent.futures
import glob
import os
import re
import shutil
import subprocess
import sysconfig
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtesseract_hip.so")
CALL_SRC = os.path.join(CSRC, "python", "tess_call.cpp")
CALL = os.path.join(HERE, "_tess_call.so")
SOURCES = sorted(glob.glob(os.path.join(CSRC, "*.cpp")) + glob.glob(os.path.join(CSRC, "*.hip")))
HEADERS = sorted(glob.glob(os.path.join(CSRC, "*.h"))) + [os.path.join(ROOT, "include", "tesseract.h"),
                                                          os.path.join(ROOT, "include", "tesseract_diag.h")]

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument",
         "-Wno-inline-asm",      # the loader's statements clobber M0 on purpose (see check_m0_writes)
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def check_m0_writes(asm_text):
    """The direct-to-LDS loader sets M0 once for a group of four requests that are issued
    at different points of the software pipeline (tess_mfma.h, DmaLoader::request).
    That is only sound if nothing else writes M0 in between, which the compiler is not
    told.  Every instruction of the generated device code whose destination is M0 must
    therefore be one of the loader's own: `s_mov_b32 m0, <sgpr>` followed by `s_nop 0`.
    Returns the list of offending lines."""
    lines = [l.strip() for l in asm_text.splitlines()]
    insns = [l for l in lines if l and not l.startswith((".", ";", "/")) and not l.endswith(":")]
    bad = []
    for i, l in enumerate(insns):
        m = re.match(r"^(\S+)\s+m0\b", l)
        if not m:
            continue
        nxt = insns[i + 1] if i + 1 < len(insns) else ""
        if not (m.group(1) == "s_mov_b32" and re.match(r"^s_nop\s+0\b", nxt)):
            bad.append(l)
    return bad


def _scalars(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand) or re.fullmatch(r"s(\d+)()", operand)
    return set(range(int(m[1]), int(m[2] or m[1]) + 1)) if m else set()


def check_request_scalars(asm_text):
    """A scalar register that a vector instruction writes may be read by a memory instruction five
    wait states later at the earliest.  The compiler keeps that distance for its own instructions
    but does not see the direct-to-LDS requests inside their asm statements: a descriptor that it
    computed in vector registers and moved over right in front of a request would be read stale,
    and the request would go to a wild address.  Returns the requests that are too near, along
    every path of up to five instructions."""
    STATES = 5
    bad, pending = set(), {}         # label -> writes still in flight where something jumps to it
    for _ in range(2):               # a second pass has the backward jumps too
        live = {}                    # scalar register -> wait states since a vector instruction wrote it
        fell = True
        for number, line in enumerate(asm_text.splitlines(), 1):
            text = line.split(";")[0].strip()
            label = re.fullmatch(r"([.\w$]+):", text)
            if label:
                if not fell:
                    live = {}
                for reg, age in pending.get(label[1], {}).items():
                    live[reg] = min(age, live.get(reg, age))
                fell = True
                continue
            if not text or text.startswith("."):
                continue
            op, _, rest = text.partition(" ")
            operands = re.findall(r"[^\s,\[]+(?:\[[^\]]*\])?", rest)
            if op.startswith("buffer_load") and operands and operands[-1] == "lds":
                used = set().union(*(_scalars(o) for o in operands))
                if any(live.get(reg, STATES) < STATES for reg in used):
                    bad.add(f"line {number}: {text}")
            step = int(operands[0], 0) + 1 if op == "s_nop" else 1
            live = {reg: age + step for reg, age in live.items() if age + step < STATES}
            if op.startswith("v_") and operands:
                # (the carry or scale result of a few instructions is their second operand)
                results = operands[:2] if re.search(r"_co_|_co_u32|v_mad_[ui]64|v_div_scale", op) else operands[:1]
                live.update({reg: 0 for o in results for reg in _scalars(o)})
            elif op.startswith("s_") and operands:
                for reg in _scalars(operands[0]):
                    live.pop(reg, None)
            if op.startswith("s_branch") or op.startswith("s_cbranch"):
                into = pending.setdefault(operands[0], {})
                for reg, age in live.items():
                    into[reg] = min(age, into.get(reg, age))
            fell = op not in ("s_branch", "s_endpgm", "s_setpc_b64")
    return sorted(bad)


def _compile(src, tmp, extra):
    """One source to an object; the device assembly is kept beside it and checked."""
    stem = os.path.splitext(os.path.basename(src))[0]
    work = os.path.join(tmp, stem)
    os.mkdir(work)
    obj = os.path.join(work, stem + ".o")
    subprocess.run(["hipcc"] + FLAGS + ["--save-temps"] + list(extra) + ["-x", "hip", "-c", src, "-o", obj],
                   check=True, cwd=work)
    found = glob.glob(os.path.join(work, stem + "-hip-amdgcn*gfx950*.s"))
    if not found:
        raise RuntimeError(f"no device assembly of {src} was kept: cannot check M0 writes")
    for path in found:
        asm_text = open(path).read()
        bad = check_request_scalars(asm_text)
        if bad:
            raise RuntimeError(f"requests too near behind a vector write of their scalar registers in the device code of {src}: "
                               + "; ".join(bad[:5]))
        bad = check_m0_writes(asm_text)
        if bad:
            raise RuntimeError(f"compiler-generated writes to M0 in the device code of {src} "
                               "(they would redirect the direct-to-LDS requests): " + "; ".join(bad[:5]))
    return obj


def _compile_call(tmp):
    """The extension module: host code only, against this interpreter and the installed torch."""
    import torch
    from torch.utils import cpp_extension
    out = os.path.join(tmp, "_tess_call.so")
    includes = [os.path.join(ROOT, "include"), sysconfig.get_paths()["include"]] + cpp_extension.include_paths()
    rocm = os.path.join(os.path.dirname(os.path.realpath(shutil.which("hipcc"))), "..", "include")
    lib_dir = os.path.join(os.path.dirname(torch.__file__), "lib")
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1",
                    "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
                   + [x for i in includes + [rocm] for x in ("-isystem", i)] + [CALL_SRC, "-o", out, "-L", lib_dir]
                   + ["-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"], check=True, cwd=tmp)
    return out


def build(force=True, extra=()):
    if not force and os.path.exists(LIB) and os.path.exists(CALL):
        newest = max(os.path.getmtime(p) for p in SOURCES + HEADERS + [CALL_SRC])
        if min(os.path.getmtime(LIB), os.path.getmtime(CALL)) >= newest:
            return LIB
    with tempfile.TemporaryDirectory(prefix="tess_build_") as tmp:
        with concurrent.futures.ThreadPoolExecutor(min(len(SOURCES) + 1, os.cpu_count() or 1)) as pool:
            call = pool.submit(_compile_call, tmp)
            objs = list(pool.map(lambda src: _compile(src, tmp, extra), SOURCES))
            shutil.move(call.result(), CALL)
        out = os.path.join(tmp, "libtesseract_hip.so")
        subprocess.run(["hipcc"] + FLAGS + ["-shared"] + objs + ["-o", out], check=True, cwd=tmp)
        shutil.move(out, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
