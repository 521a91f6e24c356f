"""Build step for the gfx950 library: compiles csrc/*.hip with hipcc into
libdebyefit.so next to this file (in-tree, so the GPU machine loads exactly the
library built here)."""
import concurrent.futures as cf
import glob
import os
import re
import subprocess

_HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(_HERE, "csrc")
INC = os.path.join(os.path.dirname(_HERE), "include")
LIB = os.path.join(_HERE, "libdebyefit.so")
ARCH = os.environ.get("DEBYEFIT_ARCH", "gfx950")

COMMON = ["hipcc", f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", f"-I{INC}",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]
# per-file extra flags: the optimiser updates must be rounded operation by operation
EXTRA = {"pso.hip": ["-ffp-contract=off"], "de.hip": ["-ffp-contract=off"], "da.hip": ["-ffp-contract=off"]}
SOURCES = ["fit_ragged.hip", "fit_eval.hip", "fit_grad.hip", "fit_dd.hip", "material.hip", "swarm.hip", "pso.hip", "de.hip", "da.hip", "lbfgs.hip", "api.hip", "auto.hip",
           "noalloc.hip"]


# lane-wise instructions; lane reads and writes of scalar spills ignore the exec mask
_LANE_WISE = re.compile(r"(v_(?!readlane|writelane|readfirstlane)|scratch_|buffer_|global_|flat_|ds_)")


def masked_join_code(lines):
    """Lane-wise instructions that stand at the join of a divergent branch
    before the exec mask is restored: [(line, function, instruction)].

    Where a block starts with scalar copies or spills, hipcc's register
    allocator can take the mask's restore for the end of the block's prologue
    and put vector copies and spills ahead of it.  They then run for the lanes
    of the taken side alone, and the others go on with stale values: an adjoint
    of 11 poles that spilled 254 registers took the first weight of its last
    pass from whatever the register held before, in every lane without a
    remainder point.  No source form excludes it, so the assembly is checked."""
    found, joins = [], set()
    function, blocks = None, []

    def flush():
        for label, items in blocks:
            if label not in joins:
                continue
            ahead = []
            for n, ins in items:
                if re.match(r"s_or_b64 exec, exec|s_(or|andn2)_saveexec_b64", ins):
                    found.extend((n, function, i) for n, i in ahead)
                    break
                if re.match(r"s_cbranch|s_branch|s_endpgm|s_setpc|s_and_saveexec|s_and_b64 exec|s_andn2_b64 exec", ins):
                    break
                if _LANE_WISE.match(ins):
                    ahead.append((n, ins))

    for n, line in enumerate(lines, 1):
        label = re.match(r"(\.LBB\w+|\w+):", line)
        if label and not label[1].startswith(".LBB"):
            flush()
            function, blocks, joins = label[1], [], set()
            continue
        if label or line.startswith("; %bb."):
            blocks.append((label[1] if label else None, []))
            continue
        ins = line.split(";")[0].strip()
        if not blocks or not ins or ins.startswith("."):
            continue
        skip = re.match(r"s_cbranch_execz (\S+)", ins)
        if skip:
            joins.add(skip[1])
        blocks[-1][1].append((n, ins))
    flush()
    return found


def _compile(name, objdir, verbose):
    src = os.path.join(SRC, name)
    obj = os.path.join(objdir, name + ".o")
    cmd = COMMON + EXTRA.get(name, []) + ["--save-temps=obj", "-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {name}:\n{r.stderr}")
    stem = os.path.join(objdir, name[:-len(".hip")])
    asm = f"{stem}-hip-amdgcn-amd-amdhsa-{ARCH}.s"
    with open(asm) as f:
        found = masked_join_code(f)
    for temp in glob.glob(stem + "-h*") + glob.glob(obj[:-len(".o")] + "-h*"):
        if temp != asm:
            os.remove(temp)
    if found:
        raise RuntimeError(f"{name}: lane-wise code ahead of a mask's restore ({len(found)}): {found[:8]}")
    return obj


def build(verbose=False, jobs=None):
    objdir = os.path.join(_HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    jobs = jobs or min(len(SOURCES), os.cpu_count() or 4)
    with cf.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(lambda n: _compile(n, objdir, verbose), SOURCES))
    tmp = LIB + ".tmp"
    cmd = ["hipcc", f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
