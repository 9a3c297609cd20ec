"""Build liblvx.so (the C-ABI HIP library) for gfx950, in-tree, with hipcc.

    python -m paper_2502_02406_amd.build

Every translation unit under csrc/ is compiled with
``hipcc --offload-arch=gfx950 -O3`` and linked into ``paper_2502_02406_amd/liblvx.so``.
hipcc cross-compiles, so this runs on machines without a GPU.
"""
from __future__ import annotations

import glob
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "liblvx.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         # hipcc may fuse scalar float math into packed-fp32 instructions; keep them off
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument",
         # the tile-copy statements name m0 as clobbered on purpose (they load it with the LDS
         # address); clang notes for every use that it does not preserve a reserved register
         "-Wno-inline-asm"]


# Per-file flags.  The key-stationary backward kernel runs one wave per SIMD with the whole
# register file; there the compiler would by default put every matrix-instruction result into the
# accumulation registers, including the scores that the vector ALU consumes next.  Its own
# accumulators are pinned to that file in the source, everything else stays in ordinary registers.
FILE_FLAGS = {"lvx_bwd_dkdv_bf16.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
              # (two or three waves per SIMD: one file of 256 or 168 registers instead of two halves)
              "lvx_bwd_dkdv_short_bf16.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
              # (its contraction phase is one unrolled run of 48 matrix instructions with the vector work
              # of a step between them: larger than what the unroll pragma accepts by default)
              "lvx_bwd_fused_bf16.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1",
                                         "-mllvm", "-pragma-unroll-threshold=200000"]}


# Kernels whose accumulators are registers that their statements name (lvx_tile_run.h).  The compiler does not know that these hold
# anything, so the code that it made is looked at, here, where another compiler that uses one of them would otherwise
# make a library with wrong projections.
NAMED_ACCUMULATORS = {"lvx_project.hip": "project_run_bf16_kernel", "lvx_project_bwd.hip": "project_bwd_x_run_bf16_kernel"}


def check_named_accumulators(asm: str, kernel: str) -> None:
    """Raises unless, in both instantiations of the kernel, the accumulation registers a0 .. a255 are the 16 blocks of its matrix
    instructions and nothing else: a block is started from 0 or added to, its operands are ordinary registers, every register is read
    for each of the two places that pack a finished tile, and there is no spill."""
    bodies = re.findall(r"^_ZN[^\n]*" + kernel + r"[^\n]*:[^\n]*\n(.*?)^\.Lfunc_end\d+:", asm, re.S | re.M)
    if len(bodies) != 2:
        raise RuntimeError(f"{kernel}: {len(bodies)} instantiations in the generated code, not 2")
    def block(op):                                   # a[16 B:16 B + 15] -> B
        m = re.fullmatch(r"a\[(\w+):(\w+)\]", op)
        first, last = (int(m[1], 0), int(m[2], 0)) if m else (-1, -1)
        return first // 16 if m and first % 16 == 0 and last == first + 15 else None

    for body in bodies:
        started, added, reads = set(), set(), []
        for line in body.splitlines():
            name, _, rest = line.split(";")[0].strip().partition(" ")
            ops = [o.strip() for o in rest.split(",")]
            used = any(re.match(r"a(\d+$|\[)", o) for o in ops)
            ok = not name.startswith("scratch_")
            if name == "v_mfma_f32_32x32x16_bf16":
                ok = (block(ops[0]) is not None and all(re.fullmatch(r"v\[\d+:\d+\]", o) for o in ops[1:3])
                      and (ops[3] == "0" or block(ops[3]) == block(ops[0])))
                (started if ops[3] == "0" else added).add(block(ops[0]))
            elif name == "v_accvgpr_read_b32":
                m = re.fullmatch(r"a\[(\w+)\]", ops[1])
                ok = m is not None and re.fullmatch(r"v\d+", ops[0]) is not None
                reads.append(int(m[1], 0) if m else None)
            elif used or name.startswith(("v_accvgpr", "v_mfma")):
                ok = False
            if not ok:
                raise RuntimeError(f"{kernel}: the named accumulators are used elsewhere: {line.strip()}")
        if started != set(range(16)) or added != set(range(16)) or sorted(reads) != sorted(2 * list(range(256))):
            raise RuntimeError(f"{kernel}: blocks started {sorted(started)}, added to {sorted(added)}, {len(reads)} reads")


def _check_generated(src: str, obj: str) -> None:
    """Looks at the code of an object that was compiled with its intermediate files kept, and removes these."""
    made = [f for f in glob.glob(obj[:-2] + "[-.]*") if f != obj]
    asm = [f for f in made if f.endswith("-gfx950.s")]
    try:
        if len(asm) != 1:
            raise RuntimeError(f"no generated code of {src} found")
        with open(asm[0]) as f:
            check_named_accumulators(f.read(), NAMED_ACCUMULATORS[os.path.basename(src)])
    except Exception:
        os.remove(obj)
        raise
    finally:
        for f in made:
            os.remove(f)


def _compile(src: str, force: bool, extra) -> str:
    obj = os.path.join(OBJ, os.path.basename(src).replace(".hip", ".o"))
    deps = [src] + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(HERE, "..", "include", "*.h"))
    if not force and os.path.exists(obj) and all(os.path.getmtime(obj) >= os.path.getmtime(d) for d in deps):
        return obj
    look = os.path.basename(src) in NAMED_ACCUMULATORS
    cmd = [HIPCC] + FLAGS + FILE_FLAGS.get(os.path.basename(src), []) + list(extra) + ["-c", src, "-o", obj] + \
        (["--save-temps=obj"] if look else [])
    r = subprocess.run(cmd, capture_output=True, text=True)
    msgs = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                     if "packed-fp32-ops" not in l and l.strip())
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{msgs}")
    if msgs:
        print(msgs, file=sys.stderr)
    if look:
        _check_generated(src, obj)
    return obj


def build(force: bool = True, extra_flags=(), output: str = None) -> str:
    """Compile every csrc/*.hip for gfx950 and link liblvx.so; returns its path.  With `output`
    the library goes to that path instead (a variant built with other definitions, to be loaded
    through the LVX_LIB environment variable), its objects into a directory of their own."""
    global OBJ
    lib, obj_dir = LIB, OBJ
    if output:
        lib = os.path.abspath(output)
        OBJ = os.path.join(obj_dir, "variant_" + os.path.basename(lib).replace(".", "_"))
    try:
        os.makedirs(OBJ, exist_ok=True)
        srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
        with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
            objs = list(ex.map(lambda s: _compile(s, force, extra_flags), srcs))
    finally:
        OBJ = obj_dir
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib] + objs
    subprocess.run(cmd, check=True)
    return lib


if __name__ == "__main__":
    # --define NAME=VALUE (repeatable): extra preprocessor definitions, e.g. the measurement switches
    # of the fused backward kernel
    # --output PATH: link the library there instead of replacing liblvx.so
    defs = [f"-D{sys.argv[i + 1]}" for i, a in enumerate(sys.argv[:-1]) if a == "--define"]
    outs = [sys.argv[i + 1] for i, a in enumerate(sys.argv[:-1]) if a == "--output"]
    print(build(force="--incremental" not in sys.argv or bool(defs), extra_flags=defs,
                output=outs[-1] if outs else None))
