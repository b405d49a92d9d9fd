"""Build libndvm.so in-tree for gfx950 with hipcc.

Kernels and host code are compiled with -ffp-contract=off (no implicit fused
multiply-add: every +, -, *, / is one IEEE operation, matching the oracle)
and with packed-fp32 instructions disabled.
"""
from __future__ import annotations

import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libndvm.so")
# host emulator of device programs: a scheduler-checking tool loaded only by the CPU tests
EMU_OUT = os.path.join(HERE, "libndvm_emu.so")
BUILD = os.path.join(HERE, "_build")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

SOURCES = ["frontend.cpp", "tape.cpp", "sched.cpp", "wide_sched.cpp", "abi.cpp", "kernels.hip", "wide.hip", "optim.hip",
           "walk_host.cpp", "walk.hip"]
EMU_SOURCES = ["frontend.cpp", "tape.cpp", "sched.cpp", "wide_sched.cpp", "emu.cpp"]
COMMON = ["-O3", "-fPIC", "-std=c++17", "-ffp-contract=off", "-fno-fast-math", "-Wall",
          "-Wno-unused-function"]
DEVICE = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# the replay kernel's options
REPLAY = [
    # the interpreter's dispatch branches are wave-uniform: leave such
    # regions unstructured instead of routing every handler exit through a
    # chain of flow blocks
    "-mllvm", "-structurizecfg-skip-uniform-regions=true",
    # keep every handler's final register store in the handler: sunk into a
    # shared block it would wait there for the memory traffic of every other
    # handler (the program prefetch included)
    "-mllvm", "-sink-common-insts=false", "-mllvm", "-enable-tail-merge=false"]
# sources built with the replay kernel's options
REPLAY_OPTIONS_FOR = {"wide_sched.cpp", "frontend.cpp", "tape.cpp", "sched.cpp", "abi.cpp", "kernels.hip", "optim.hip", "emu.cpp",
                      "walk.hip"}

# The walker's loop: without lifetime markers leaving a handler's scope is a
# plain branch, not a value tested by a chain of blocks behind every handler.
WALK = ["-Xclang", "-disable-lifetime-markers"]

# The wide kernel: the library functions' branches on wave-uniform values stay
# branches; the registers its inline asm names are not the compiler's.
WIDE = ["-mllvm", "-structurizecfg-skip-uniform-regions=true", "-Wno-inline-asm"]



def _options(src: str) -> list:
    extra = REPLAY if src in REPLAY_OPTIONS_FOR else WIDE if src == "wide.hip" else []
    return COMMON + DEVICE + extra + (WALK if src == "walk.hip" else [])


# Library functions that inline asm calls past their first instruction, which has
# to be a wait of 4 bytes, and the registers they may use: (vector below,
# scalar below, scalar besides) by name.
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
_WIDE_SCALAR = "exp sin cos logc sqrtc pow accsin acccos acclog accabs accpow accsqrt abs".split()
_WIDE_MATRIX = ("mm mma mmb vadd vacc trans transacc inv2 inv2acc vscale vaccs sdot det2 "
                "logdetacc").split()
CALLED = {
    "wide.hip": {**{"ndvm_wide_" + f: (39, 26, {30, 31}) for f in _WIDE_SCALAR},
                 **{"ndvm_wide_" + f: (95, 26, {27, 30, 31}) for f in _WIDE_MATRIX}},
    "walk.hip": {"ndvm_walk_" + f: (40, 32, set()) for f in ("sin", "cos", "pow")}}


def check_called(src: str, listing: str) -> None:
    """Raise unless each function of CALLED[src] in the disassembly begins with
    that wait and keeps to its registers, without scratch memory or calls."""
    body = {}
    for line in listing.splitlines():
        m = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if m:
            body[m.group(1)] = cur = []
        m = re.match(r"\s+(.*?)\s+// [0-9A-F]+: ([0-9A-F ]+)", line)
        if m:
            cur.append((m.group(1), len(m.group(2).split()) * 4))
    for f, (vector, scalar, besides) in CALLED[src].items():
        code = body.get(f, [])
        if not code or code[0] != ("s_waitcnt vmcnt(0) expcnt(0) lgkmcnt(0)", 4):
            raise RuntimeError(f"{src}: {f} does not begin with the wait that its calls skip: {code[:1]}")
        for text, _ in code:
            if re.search(r"scratch|buffer|\bm0\b|swappc", text):
                raise RuntimeError(f"{src}: {f} uses what its callers do not provide: {text}")
            for kind, lo, hi, one in re.findall(r"\b([sv])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
                for r in range(int(lo or one), int(hi or one) + 1):
                    if r >= (scalar if kind == "s" else vector) and not (kind == "s" and r in besides):
                        raise RuntimeError(f"{src}: {f} uses {kind}{r}, which its callers hold: {text}")


def _check(src: str) -> None:
    obj = os.path.join(BUILD, "device_" + os.path.splitext(src)[0] + ".o")
    subprocess.run([HIPCC] + _options(src) + ["--cuda-device-only", "--no-gpu-bundle-output", "-c",
                                              os.path.join(CSRC, src), "-o", obj], check=True, capture_output=True)
    check_called(src, subprocess.run([OBJDUMP, "-d", obj], check=True, capture_output=True, text=True).stdout)


# The emulator's copies of the sources check every element access of the
# standard containers (the process ends at one out of range).
EMU = ["-D_GLIBCXX_ASSERTIONS"]


def _compile(src: str, emu: bool = False) -> str:
    obj = os.path.join(BUILD, ("emu_" if emu else "") + os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + _options(src) + (EMU if emu else []) + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in (r.stderr or "").splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _link(objs, out):
    tmp = out + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}"] + objs + ["-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, out)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    jobs = [(s, False) for s in SOURCES] + [(s, True) for s in EMU_SOURCES]
    with ThreadPoolExecutor(max_workers=len(jobs) + len(CALLED)) as ex:
        checks = [ex.submit(_check, s) for s in CALLED]
        objs = list(ex.map(lambda j: _compile(*j), jobs))
        for c in checks:
            c.result()
    _link(objs[:len(SOURCES)], OUT)
    _link(objs[len(SOURCES):], EMU_OUT)
    if verbose:
        print("built", OUT, "and", EMU_OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
