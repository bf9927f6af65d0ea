"""Builds libptq.so (the C-ABI library of hand-written gfx950 kernels) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libptq.so")
PROBE_LIB = os.path.join(HERE, "libptq_probe.so")   # diagnostics for bench.py --mfma-control, not part of the product
SOURCES = ["ptq_api.hip", "hessian.hip", "hessian_f32.hip", "cholesky.hip", "quantize.hip", "vq.hip", "layer_error.hip", "lopro.hip", "r1svd.hip", "r1svd_bf16.hip", "artifact.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-result",
    # packed-FP32 instructions are kept out of every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]
# Accumulators of the float64 matrix instructions stay in ordinary VGPRs (those kernels fit
# 256 registers, and the AGPR form costs copies around each MFMA).  The bf16 Hessian kernel
# needs all 256 AGPRs for its accumulators and is compiled without the option.
VGPR_FORM = ["-mllvm", "-amdgpu-mfma-vgpr-form"]
NO_VGPR_FORM = {"hessian.hip"}


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    raise RuntimeError("hipcc not found")


def check_dpp_wait_states(asm_text: str) -> int:
    """The leaf of cholesky.hip's factor issues DPP instructions from inline assembly, where the compiler
    does not count wait states: a DPP read needs two (two instructions, or s_nop) after a vector
    instruction wrote the register it reads.  The source keeps that distance by construction; this walks
    the generated assembly and raises if the compiler has put something closer (a copy into an
    accumulator, say).  Returns the number of DPP instructions seen."""
    import re

    def regs(tok):
        m = re.match(r"v\[(\d+):(\d+)\]", tok)
        if m:
            return set(range(int(m.group(1)), int(m.group(2)) + 1))
        m = re.match(r"v(\d+)$", tok)
        return {int(m.group(1))} if m else set()

    lines = [l.strip() for l in asm_text.splitlines()]
    lines = [l for l in lines if l and not l.startswith((";", ".")) and not l.endswith(":")]
    seen = 0
    for i, l in enumerate(lines):
        if "row_newbcast" not in l:
            continue
        seen += 1
        src0 = regs(l.split(None, 1)[1].split(",")[1].split()[0])
        waited, k = 0, i - 1
        while waited < 2 and k >= 0:
            p = lines[k]
            m = re.match(r"s_nop (\d+)", p)
            if m:
                waited += int(m.group(1)) + 1
            else:
                if p.startswith("v_") and regs(p.split(None, 1)[1].split(",")[0].split()[0]) & src0:
                    raise RuntimeError(f"DPP read too close to the write of its source:\n  {p}\n  {l}")
                waited += 1
            k -= 1
    return seen


def check_lds_dma_wait_states(asm_text: str) -> int:
    """lds_dma.h issues its loads into LDS from inline assembly, where the compiler does not count wait states: such a load
    needs one after a scalar instruction wrote m0, and five after a vector instruction wrote a scalar register of its
    operands.  Walks the generated assembly back from every such load, into all predecessors at a label, and raises
    if something stands closer.  Returns the number of loads seen."""
    import re

    def sgprs(tok):
        m = re.match(r"s\[(\d+):(\d+)\]$", tok)
        if m:
            return set(range(int(m.group(1)), int(m.group(2)) + 1))
        m = re.match(r"s(\d+)$", tok)
        return {int(m.group(1))} if m else ({"vcc"} if tok == "vcc" else set())

    lines = [l.split(";")[0].strip() for l in asm_text.splitlines()]
    lines = [l for l in lines if l and (not l.startswith(".") or re.match(r"\.\w+:$", l))]
    jumps = {}   # label -> the branches to it
    for i, l in enumerate(lines):
        m = re.match(r"s_c?branch\S* (\S+)$", l)
        if m:
            jumps.setdefault(m.group(1), []).append(i)

    def walk(i, left, load, operands, adjacent):
        """From line i back while `left` wait states are missing."""
        while left > 0 and i >= 0:
            l = lines[i]
            if l.endswith(":"):
                for j in jumps.get(l[:-1], []):
                    walk(j, left, load, operands, adjacent)
                if i > 0 and re.match(r"s_(branch|endpgm|setpc)", lines[i - 1]):
                    return
                i -= 1
                continue
            toks = re.split(r"[ ,]+", l)
            if toks[0] == "s_nop":
                left -= int(toks[1], 0) + 1
                adjacent = False
            else:
                wrote = toks[1] if len(toks) > 1 else ""
                if adjacent and wrote == "m0":
                    raise RuntimeError(f"load into LDS directly after the write of m0:\n  {l}\n  {load}")
                if toks[0].startswith("v_") and sgprs(wrote) & operands:
                    raise RuntimeError(f"load into LDS too close to the write of its scalar operand:\n  {l}\n  {load}")
                left -= 1
                adjacent = False
            i -= 1

    seen = 0
    for i, l in enumerate(lines):
        if l.startswith(("buffer_load", "global_load")) and re.search(r"\blds$", l):
            seen += 1
            walk(i - 1, 5, l, set().union(*(sgprs(t) for t in re.split(r"[ ,]+", l)[1:])), True)
    return seen


# what is checked on a source's generated assembly
ASSEMBLY_CHECKS = {
    "cholesky.hip": check_dpp_wait_states,
    "hessian.hip": check_lds_dma_wait_states,
    "layer_error.hip": check_lds_dma_wait_states,
    "artifact.hip": check_lds_dma_wait_states,
}


def device_assembly(src: str) -> str:
    extra = [] if src in NO_VGPR_FORM else VGPR_FORM
    cmd = [_hipcc(), *[f for f in FLAGS if f not in ("-fPIC", "-Wall")], *extra, "-S", "--cuda-device-only",
           os.path.join(CSRC, src), "-o", "-"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc -S failed for {src}:\n{r.stderr}")
    return r.stdout


def check_assembly(src: str) -> None:
    if ASSEMBLY_CHECKS[src](device_assembly(src)) == 0:
        raise RuntimeError(f"{src}: none of the checked instructions found in the generated assembly (check out of date?)")


def build(verbose: bool = True) -> str:
    """Compiles every source (always, also when a library is already there) and links."""
    hipcc = _hipcc()
    objs = []

    def compile_one(src):
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        extra = [] if src in NO_VGPR_FORM else VGPR_FORM
        cmd = [hipcc, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
        errs = [l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip()]
        if verbose and any("warning" in l for l in errs):
            print("\n".join(errs), file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=8) as ex:
        checked = [ex.submit(check_assembly, src) for src in ASSEMBLY_CHECKS]
        objs = list(ex.map(compile_one, SOURCES))
        for c in checked:
            c.result()
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    # the register-only MFMA probe, a library of its own: one source, compiled in both accumulator forms
    probe_objs = []
    for tag, extra in (("agpr", []), ("vgpr", ["-DPTQ_PROBE_VGPR_FORM", *VGPR_FORM])):
        obj = os.path.join(CSRC, f"probe_mfma_{tag}.o")
        r = subprocess.run([hipcc, *[f for f in FLAGS if f != "-Wall"], *extra, "-c", os.path.join(CSRC, "probe_mfma.hip"),
                            "-o", obj], capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"probe library failed:\n{r.stdout}\n{r.stderr}")
        probe_objs.append(obj)
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", PROBE_LIB, *probe_objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"probe library failed:\n{r.stdout}\n{r.stderr}")
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
