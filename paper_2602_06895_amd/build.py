"""Build libmsx.so (HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmsx.so")
# the six chain_*.hip units (register class x precision) are the slow ones and
# compile in parallel with the rest
SOURCES = ["chain_f64_l.hip", "chain_f64_m.hip", "chain_f64_s.hip", "chain_mix_l.hip", "chain_mix_m.hip",
           "chain_mix_s.hip", "kernels.hip", "flow_kernels.hip", "flow_layers.hip", "flow_train.hip",
           "api.cpp", "flow_api.cpp", "compiler.cpp",
           "json.cpp", "jit.cpp", "inverse_s.hip", "inverse_m.hip", "inverse_l.hip"]
# headers of the fused sample kernel, compiled again at run time for a
# context's channels (jit.cpp); their text goes into the library
JIT_HEADERS = ["tables.h", "device_util.h", "chain.h", "chain_kernels.h"]
# the forward mapping chain (map, fused sample, weights) is compiled without
# floating-point contraction: every fused multiply-add is written out, so the
# class kernels and the run-time specialised sample (same flag) give
# bit-identical results; the inverse_*.hip units keep the default
NO_CONTRACT = {"chain_f64_l.hip", "chain_f64_m.hip", "chain_f64_s.hip", "chain_mix_l.hip", "chain_mix_m.hip",
               "chain_mix_s.hip", "kernels.hip"}
# Machine-level loop-invariant hoisting keeps constants and table values of the
# chain in registers over the event loop.  Without it, and with instructions
# sunk to their uses, the class kernels need 50 to 90 registers fewer (t tbar 354
# -> 256, pp -> 4 jets 247 -> 168, inverse 179 -> 128) for 1% more instructions,
# and more waves fit
FEWER_REGISTERS = {"chain_f64_l.hip", "chain_f64_m.hip", "chain_f64_s.hip", "chain_mix_l.hip", "chain_mix_m.hip",
                   "chain_mix_s.hip", "inverse_s.hip", "inverse_m.hip", "inverse_l.hip"}
ARCH = os.environ.get("MSX_OFFLOAD_ARCH", "gfx950")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         # packed FP32 instructions are never generated for this library
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include")]


def _jit_sources() -> str:
    """Writes _build/jit_sources.cpp: the kernel headers as string literals."""
    path = os.path.join(OBJ, "jit_sources.cpp")
    out = ["// Generated by build.py from the kernel headers: their text, compiled again",
           "// at run time by jit.cpp.", "namespace msx {", "namespace jit_src {",
           f"extern const int kHeaderCount = {len(JIT_HEADERS)};",
           "extern const char* const kHeaderNames[] = {" + ", ".join(f'"{h}"' for h in JIT_HEADERS) + "};",
           "extern const char* const kHeaderTexts[] = {"]
    for h in JIT_HEADERS:
        text = open(os.path.join(CSRC, h)).read()
        if ")msxsrc\"" in text:
            raise RuntimeError(f"{h} contains the raw-string delimiter")
        out.append('R"msxsrc(' + text + ')msxsrc",')
    out += ["};", "}  // namespace jit_src", "}  // namespace msx", ""]
    text = "\n".join(out)
    if not os.path.exists(path) or open(path).read() != text:
        with open(path, "w") as f:
            f.write(text)
    return path


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(os.path.basename(src))[0] + ".o")
    path = src if os.path.isabs(src) else os.path.join(CSRC, src)
    flags = FLAGS + (["-ffp-contract=off"] if src in NO_CONTRACT else []) + ["-I", CSRC]
    if src in FEWER_REGISTERS:
        flags += ["-mllvm", "-disable-machine-licm", "-mllvm", "-sink-insts-to-avoid-spills"]
    cmd = [HIPCC] + flags + ["-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    """Compile every source and link libmsx.so (always rebuilds)."""
    os.makedirs(OBJ, exist_ok=True)
    workers = max(1, min(len(SOURCES), int(os.environ.get("MAX_JOBS", os.cpu_count() or 4))))
    with ThreadPoolExecutor(max_workers=workers) as ex:
        objs = list(ex.map(_compile, SOURCES + [_jit_sources()]))
    tmp = LIB + ".tmp%d" % os.getpid()
    rocm_lib = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(HIPCC))), "lib")
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp] + objs + [
        "-L" + rocm_lib, "-lhiprtc", "-Wl,-rpath," + rocm_lib]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
