"""Builds libavq.so (HIP, gfx950 only) in-tree with hipcc.

`python -m paper_1908_10396_amd.build` compiles every translation unit under
csrc/ and links them into paper_1908_10396_amd/libavq.so. hipcc cross-compiles
for gfx950 without a GPU present.
"""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libavq.so")
UNITS = ["api", "lut", "scan", "scan_mfma", "product", "product_leaf", "refine", "select", "ivf", "layout", "nearest", "exact", "train"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17",
    "-ffp-contract=off",                      # the fp32 query path has a defined operation order
    "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def _newer(target, sources):
    if not os.path.exists(target):
        return False
    t = os.path.getmtime(target)
    return all(os.path.getmtime(s) <= t for s in sources)


SHIFT64 = re.compile(r"\s*v_(?:lshlrev_b64|lshrrev_b64|ashrrev_i64)(?:_e64)?\s+v\[\d+:\d+\],\s*v(\d+),")
LSHL_ADD64 = re.compile(r"\s*v_lshl_add_u64(?:_e64)?\s+v\[\d+:\d+\],\s*[^,]+,\s*v(\d+),")
VGPR = re.compile(r"\bv(?:(\d+)\b|\[\d+:(\d+)\])")


def shifts_by_last_register(asm):
    """The functions of the device assembly (its lines) that shift a 64-bit value by an amount in their last vector register.

    Vector registers are allocated in eights. A 64-bit vector shift whose amount lies in the last one of the allocation
    has taken v0, the thread's index, as its amount now and then on MI355X, in one wave of sixteen that run the same
    instruction: leaf_top_kernel (48 registers) had `v_lshlrev_b64 v[28:29], v47, -1` behind a barrier, and up to half of its
    selections among many equal scores were wrong. Replaying the selection on the CPU with that one shift taken by the lane's
    index instead gives every wrong threshold that was recorded, to the digit. (The compiler knows the case for another
    target of the same family and avoids it there.) A scalar amount, or one in a lower register, is not affected."""
    bad, name, amounts, top = [], None, [], -1

    def close():
        if any((a + 1) % 4 == 0 and a >= top for a in amounts):  # (fours: where accumulation registers begin)
            bad.append(name)

    for line in asm:
        if line.startswith("_Z") and ":" in line:
            close()
            name, amounts, top = line.split(":")[0], [], -1
            continue
        code = line.split(";")[0]
        m = SHIFT64.match(code) or LSHL_ADD64.match(code)
        if m:
            amounts.append(int(m.group(1)))
        for one, last in VGPR.findall(code):
            top = max(top, int(one or last))
    close()
    return sorted(set(bad))


def build(force=True, verbose=False, jobs=8):
    os.makedirs(OBJ, exist_ok=True)
    headers = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    headers.append(os.path.join(os.path.dirname(HERE), "include", "avq.h"))
    hipcc = _hipcc()

    def compile_one(u):
        src = os.path.join(CSRC, u + ".hip")
        obj = os.path.join(OBJ, u + ".o")
        if not force and _newer(obj, [src] + headers):
            return obj
        # -save-temps=obj leaves the device assembly beside the object: it is checked below, then the extras go
        cmd = [hipcc] + FLAGS + ["-save-temps=obj", "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (u, r.stdout, r.stderr))
        if verbose and r.stderr.strip():
            print(r.stderr, file=sys.stderr)
        _check_device_code(u)
        return obj

    def _check_device_code(u):
        asm = os.path.join(OBJ, u + "-hip-amdgcn-amd-amdhsa-gfx950.s")
        with open(asm) as f:
            bad = shifts_by_last_register(f)
        for f in os.listdir(OBJ):
            if f.startswith(u + "-hip-") or f.startswith(u + "-host-") or f.startswith(u + ".hip-"):
                os.remove(os.path.join(OBJ, f))
        if bad:
            raise RuntimeError("%s.hip: a 64-bit shift by the last vector register in %s" % (u, ", ".join(bad)))

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(compile_one, UNITS))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    return LIB


if __name__ == "__main__":
    print(build(force="--incremental" not in sys.argv, verbose=True))
