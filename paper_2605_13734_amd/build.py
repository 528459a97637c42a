"""Build libkvc.so for gfx950 with hipcc (cross-compiles without a GPU).

After compiling, the device assembly of every kernel is checked for one instruction form that this
GPU executes wrongly and this compiler does not avoid for gfx950: a 64-bit shift (v_lshlrev_b64,
v_lshrrev_b64, v_ashrrev_i64) whose shift count is the last VGPR of the wave's allocation (register
number 8n+7 with no allocated register after it).  Four waves per SIMD of a kernel with
`v_lshlrev_b64 v[a:b], v111, v[c:d]` and 112 registers shifted by the lane number instead of the
count in about one execution of eight (a stand-alone kernel that does nothing else shows it; with
120 registers allocated, or the count in v109, it never does).  LLVM describes and works around
the same fault for gfx90a only.  A kernel that trips the check gets register headroom: an empty
asm statement naming a higher register (see decode_kernel).

The assembly is also searched for scalar loads at places that are no multiple of four.  Scalar loads drop the two
lowest bits of the base and of the offset, each by itself, and the compiler does not know: with a 16-bit member between the words of a
kernel's arguments, indexed at run time, it took the address of a word apart into a base two bytes too far and an offset of -2, and the
kernel read half of each of two pointers (and faulted).  A kernel's arguments have members of whole words only (CoderBatch).

A second check keeps kernels whose time depends on their waves (min_waves in kvc_quant.hip) within the
registers that leave room for them, a third one looks for rows that are requested and waited for one at a time
(rows_requested in kvc_tile.h).
"""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
OUT = os.path.join(HERE, "libkvc.so")
WIDTHS = (2, 3, 4, 8)
# (source, code width or None): the kernel sources are compiled once per code width, which spreads
# the build over the cores; the slowest units come first
JOBS = ([("kvc_huff_enc.hip", b) for b in WIDTHS] + [("kvc_quant.hip", b) for b in WIDTHS] +
        [("kvc_huff_dec.hip", b) for b in WIDTHS] +
        [("kvc_huff_tables.hip", None), ("kvc_selftest.hip", None), ("kvc_service.hip", None), ("kvc_probe.hip", None),
         ("kvc_api.hip", None), ("kvc_policy.hip", None)])
# packed fp32 instructions are switched off for the device pass (flag for hipcc only); host functions may take 44 KB of stack, which
# the calls need for the items of a full window (they run on threads of other programs)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall",
         "-Xarch_host", "-Wframe-larger-than=45056", "-Xarch_host", "-Werror=frame-larger-than", "-Wno-unused-command-line-argument"]


def shift_count_in_last_vgpr(asm_path):
    """[(kernel symbol, instruction)] for 64-bit shifts that take their count from the last
    allocated VGPR, read from the device assembly hipcc leaves with -save-temps."""
    text = open(asm_path).read()
    next_free = {k: int(re.search(r"\.amdhsa_next_free_vgpr (\d+)", body).group(1))
                 for k, body in re.findall(r"\.amdhsa_kernel (\w+)\n(.*?)\.end_amdhsa_kernel", text, re.S)}
    shift = re.compile(r"\s+v_(?:lshlrev_b64|lshrrev_b64|ashrrev_i64)\s+v\[\d+:\d+\],\s*v(\d+),")
    hits, cur = [], None
    for line in text.split("\n"):
        m = re.match(r"^(\w+):", line)
        if m and m.group(1) in next_free:
            cur = m.group(1)                         # a kernel's code starts at its symbol ...
        elif line.startswith(".Lfunc_end"):
            cur = None                               # ... and ends here
        elif cur is not None:
            m = shift.match(line)
            if m and int(m.group(1)) % 8 == 7 and int(m.group(1)) + 1 >= next_free[cur]:
                hits.append((cur, line.strip()))
    return hits


def scalar_loads_off_words(asm_path):
    """[(function or kernel symbol, instruction)] for scalar loads whose offset is no multiple of four."""
    load = re.compile(r"\s+s_(?:buffer_)?load_dword\w*\s+(.*)")
    hits, cur = [], None
    for line in open(asm_path).read().split("\n"):
        m = re.match(r"^(\w+):", line)
        if m:
            cur = m.group(1)
        m = load.match(line.split(";")[0])
        if m and any(int(n, 0) % 4 for n in re.findall(r"(?:,\s*|offset:)(-?(?:0x[0-9a-f]+|\d+))\b", m.group(1))):
            hits.append((cur, line.strip()))
    return hits


def spilling_kernels(asm_path):
    """[(kernel symbol, scratch bytes per lane)] of the kernels that spill registers."""
    text = open(asm_path).read()
    out = []
    for k, body in re.findall(r"\.amdhsa_kernel (\w+)\n(.*?)\.end_amdhsa_kernel", text, re.S):
        n = int(re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", body).group(1))
        if n:
            out.append((k, n))
    return out


# (kernel symbol, registers): six waves per SIMD for the compress kernels of one pass for bf16 rows that are not
# dense, five for 8-bit codes.  Decoders below 8 bits: four, but for two kinds with short runs of the delta transform and fp16 (4 bits dense,
# 3 bits V strided).
# Encoders: three for dense K blocks of 64 bf16 rows with the delta transform.
REGISTERS = [(r"decode_kernelILi[234]ELi\dELi\dELb\dELi[012]E", 128), (r"decode_kernelILi(?!4ELi1ELi\dELb1|3ELi1ELi1ELb0)[234]ELi\dELi\dELb\dELi3E", 128),
             (r"encode_kernelILi[234]ELi64ELi2ELi0ELb1ELb1ELi4E", 168),
             (r"compress_(?:k_kernelILi[234]ELi32|v_kernelILi[234]ELi\d+)ELi2ELb0E", 80),
             (r"compress_(?:k_kernelILi8ELi32|v_kernelILi8ELi\d+)ELi2ELb0E", 96)]


def over_budget(asm_path):
    """[(kernel symbol, registers, budget)] of the kernels that need more registers than REGISTERS gives them."""
    text = open(asm_path).read()
    out = []
    for k, body in re.findall(r"\.amdhsa_kernel (\w+)\n(.*?)\.end_amdhsa_kernel", text, re.S):
        n = int(re.search(r"\.amdhsa_next_free_vgpr (\d+)", body).group(1))
        out += [(k, n, most) for pattern, most in REGISTERS if re.search(pattern, k) and n > most]
    return out


# (kernel symbol, scalars): scalar registers that the coder's kernels may move to vector registers and back: in encoders with the delta
# transform a few (8-bit encoders as many as they do)
SCALARS = [(r"decode_kernelILi", 0), (r"encode_kernelILi[234]ELi\d+ELi\dELi\dELb\dELb0E", 0), (r"encode_kernelILi[234]", 16)]


def scalar_spills(asm_path):
    """[(kernel symbol, scalars, most)] of the kernels that spill more scalar registers than SCALARS has it."""
    text = open(asm_path).read()
    out = []
    for k, n in re.findall(r"\.name:\s+(\w+)\n(?:(?!\.name:).*\n)*?\s+\.sgpr_spill_count:\s*(\d+)", text):
        for pattern, most in SCALARS:
            if re.search(pattern, k):
                out += [(k, int(n), most)] * (int(n) > most)
                break
    return out


# (kernel symbol, most such waits): dense rows without the delta transform.  The codec-free K kernels have one at their start (the
# head list); the encoders have nine more (tables, samples and places), behind which no row is loaded.  Rotated K blocks of 64 and 128 strided fp16 rows: the
# look-ups of their pages, as without the rotation.
LONE_LOADS = [(r"compress_k_kernelILi\d+ELi64ELi1ELb0ELi2E", 18), (r"compress_k_kernelILi\d+ELi128ELi1ELb0ELi2E", 34),
              (r"encode_kernelILi\d+ELi64ELi1ELi0ELb0ELb0ELi\dELb1E", 26), (r"encode_kernelILi\d+ELi128ELi1ELi0ELb0ELb0ELi\dELb1E", 40),
              (r"compress_k_kernelILi(?!8ELi128ELi1ELb1ELi2E)\d+ELi\d+ELi\dELb1ELi[02]E", 1),
              (r"encode_kernelILi\d+ELi\d+ELi\dELi[01]ELb1ELb0E", 10)]


def lone_loads(asm_path):
    """[(kernel symbol, waits, most)] of the kernels that wait for a single load, with none behind it in flight,
    more often than LONE_LOADS has it."""
    text = open(asm_path).read()
    out = []
    for k, body in re.findall(r"^(\w+):[^\n]*\n(.*?)^\.Lfunc_end", text, re.S | re.M):
        limits = [most for pattern, most in LONE_LOADS if re.search(pattern, k)]
        if not limits:
            continue
        loads = found = 0
        for line in body.split("\n"):
            code = line.split(";")[0]
            loads += "global_load" in code
            m = re.search(r"vmcnt\((\d+)\)", code)
            if m:
                found += m.group(1) == "0" and loads == 1
                loads = 0
        out += [(k, found, most) for most in limits if found > most]
    return out


def _compile(job):
    name, width = job
    stem = name.replace(".hip", "") + ("_b%d" % width if width else "")
    # -save-temps names its files after the source, so every job works on a copy named after itself
    src = os.path.join(OBJ, stem + ".hip")
    with open(src, "w") as f:
        f.write('#include "%s"\n' % os.path.join(SRC, name))
    obj = os.path.join(OBJ, stem + ".o")
    cmd = ["hipcc"] + FLAGS + (["-DKVC_BITS=%d" % width] if width else []) + ["-I", SRC, "-save-temps=obj", "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (name, err))
    name = stem
    asm = os.path.join(OBJ, stem + "-hip-amdgcn-amd-amdhsa-gfx950.s")
    hits = shift_count_in_last_vgpr(asm)
    if hits:
        raise RuntimeError("%s: 64-bit shift with its count in the last allocated VGPR (give the kernel register "
                           "headroom):\n%s" % (name, "\n".join("  %s: %s" % h for h in hits[:20])))
    off = scalar_loads_off_words(asm)
    if off:
        raise RuntimeError("%s: scalar loads that are not at whole words (a kernel argument with a member of fewer than four "
                           "bytes?):\n%s" % (name, "\n".join("  %s: %s" % h for h in off[:20])))
    over = over_budget(asm)
    if over:
        raise RuntimeError("%s: more registers than the kernel's waves leave room for:\n%s" % (
            name, "\n".join("  %s: %d of %d" % h for h in over[:20])))
    scalars = scalar_spills(asm)
    if scalars:
        raise RuntimeError("%s: more scalar registers spilled than allowed:\n%s" % (
            name, "\n".join("  %s: %d of %d" % h for h in scalars[:20])))
    lone = lone_loads(asm)
    if lone:
        raise RuntimeError("%s: rows waited for one at a time:\n%s" % (
            name, "\n".join("  %s: %d waits, %d allowed" % h for h in lone[:20])))
    spills = spilling_kernels(asm)
    if spills:
        err += "\n%s: %d kernels spill registers (most: %d bytes per lane): %s" % (
            name, len(spills), max(n for _, n in spills), ", ".join(k for k, _ in spills[:6]))
    for f in os.listdir(OBJ):                      # the temporaries are large and no longer needed
        if (f.startswith(stem + "-") or f.startswith(stem + ".hip-")) and f != stem + ".o":
            os.remove(os.path.join(OBJ, f))
    return obj, err


def build(verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 4)) as ex:
        results = list(ex.map(_compile, JOBS))
    if verbose:
        for _, err in results:
            if err.strip():
                print(err)
    objs = [o for o, _ in results]
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT] + objs)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
