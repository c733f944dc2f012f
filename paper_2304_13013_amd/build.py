"""Builds libswitchback.so (the gfx950 HIP kernels + C ABI) in-tree with hipcc, and its Python side with g++."""
import importlib.util
import os
import re
import shutil
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libswitchback.so")
BINDING = os.path.join(HERE, "_binding" + sysconfig.get_config_var("EXT_SUFFIX"))  # of this Python alone
SOURCES = ["quantize.hip", "gemm_i8.hip", "gemm_i8_direct.hip", "gemm_f8.hip", "gemm_bf16_tn.hip", "stable_adamw.hip", "switchback_api.hip",
           "ceilings.hip"]

# -ffp-contract=off: the quantizers and the dequantizing epilogue promise one rounding per operation.
# The packed-fp32 feature is switched off on purpose (plain v_mul/v_add/v_fma only).
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function"]


def _hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def _torch_dir():
    return os.path.dirname(importlib.util.find_spec("torch").origin)


def _torch_build():
    """The torch that the binding is compiled against, as switchback.py names the one that it runs with."""
    with open(os.path.join(_torch_dir(), "version.py")) as fh:
        text = fh.read()
    return " ".join(re.search(r"^%s = '([^']*)'" % name, text, re.M).group(1) for name in ("__version__", "git_version"))


def _build_binding():
    """csrc/binding.cpp: host code against torch's headers, no kernels.  It is handed the library's entry points when it is
    bound, and links none."""
    torch_dir = _torch_dir()
    res = subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-DSB_BUILT_FOR=\"%s\"" % _torch_build(),
                          "-isystem", os.path.join(torch_dir, "include"), "-I", sysconfig.get_paths()["include"],
                          os.path.join(CSRC, "binding.cpp"), "-o", BINDING,
                          "-L", os.path.join(torch_dir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"],
                         capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed for binding.cpp:\n%s" % res.stderr)


def check_kernels(asm):
    """Faults of a source's device assembly that no test shows reliably, as a list of texts.  The matrix-product kernels load
    LDS and memory from inline assembly, into registers that the compiler takes as written at once: a register that is spilled,
    copied or reused while its load is on the way holds something else, and an address in it faults.  Four-wave kernels name
    their accumulators in the assembly text: a value of the compiler's in an accumulation register would be overwritten."""
    faults = []
    for entry in re.split(r"^ {2}- ", asm[asm.rfind("amdhsa.kernels:"):], flags=re.M):
        fields = dict(re.findall(r"^ +\.(name|vgpr_spill_count|private_segment_fixed_size): +(\S+)", entry, re.M))
        faults += ["%s: %s %s" % (fields.get("name"), key, value) for key, value in fields.items()
                   if key != "name" and value != "0"]
    for name, body in re.findall(r"^(\w+):(?: [^\n]*)?\n(.*?)^\.Lfunc_end", asm, re.M | re.S):
        faults += ["%s: %s (before its LDS read has landed)" % (name, line) for line in _early_uses(body)]
        if re.search(r"v_mfma_\w+ a\[\d+:\d+\], v\S+ v\S+ 0", body):  # an accumulator named in the text, cleared
            code = re.sub(r";;#ASMSTART\n.*?;;#ASMEND", "", body, flags=re.S)
            faults += ["%s: %s" % (name, line.strip()) for line in code.splitlines()
                       if re.search(r"\ba\d+\b|\ba\[", line.split(";")[0])]
    return faults


def _early_uses(body):
    """Instructions of a kernel that touch a register whose LDS read has not been waited for, on any way through it."""
    def registers(text):  # a bit each
        mask = 0
        for first, last, single in re.findall(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", text):
            mask |= 1 << int(single) if single else (1 << int(last) + 1) - (1 << int(first))
        return mask

    # Blocks of steps: touch registers; wait until at most so many LDS operations are on the way; start one that will write
    # these registers (none: a write, a scalar load); go to a label, and perhaps on; end.
    blocks, labels = [[]], {}
    for line in body.splitlines():
        line = line.split(";")[0].strip()
        label = re.match(r"(\.LBB\w+):$", line)
        if label:
            labels[label.group(1)] = len(blocks)
            blocks.append([])
        if not line or line[0] == "." or line[-1] == ":":
            continue
        op, _, rest = line.partition(" ")
        steps = blocks[-1]
        if op == "s_waitcnt":
            count = re.search(r"lgkmcnt\((\d+)\)", rest)
            if count:
                steps.append(("wait", int(count.group(1)), line))
        elif op in ("s_branch", "s_endpgm") or op.startswith("s_cbranch"):
            steps.append((op, rest.strip(), line))
        else:
            touched = registers(rest)
            if touched:
                steps.append(("touch", touched, line))
            if op.startswith("ds_read"):
                steps.append(("start", registers(rest.split(",")[0]), line))
            elif op.startswith(("ds_", "s_load", "s_buffer_load")):
                steps.append(("start", 0, line))
    found, seen, todo = {}, set(), [(0, ())]
    while todo:
        state = todo.pop()
        if state in seen or state[0] >= len(blocks):
            continue
        seen.add(state)
        index, flying = state
        for kind, what, line in blocks[index]:
            if kind == "touch":
                if any(what & f for f in flying):
                    found[line] = True
            elif kind == "wait":
                flying = flying[len(flying) - what:] if 0 < what <= len(flying) else flying if what else ()
            elif kind == "start":
                flying += (what,)
            elif kind == "s_endpgm":
                break
            else:
                todo.append((labels[what], flying))
                if kind == "s_branch":
                    break
        else:
            todo.append((index + 1, flying))
    return list(found)


def build(verbose=False):
    """Compile every kernel source for gfx950, link the shared library and the Python binding.  Always recompiles."""
    out_dir = os.path.join(HERE, "_build")
    os.makedirs(out_dir, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(src):
        obj = os.path.join(out_dir, src.replace(".hip", ".o"))
        with tempfile.TemporaryDirectory() as temps:
            res = subprocess.run([hipcc, *HIPCC_FLAGS, "-save-temps=obj", "-c", os.path.join(CSRC, src), "-o",
                                  os.path.join(temps, "source.o")], capture_output=True, text=True)
            if res.returncode != 0:
                raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, res.stdout, res.stderr))
            asm, = (f for f in os.listdir(temps) if f.endswith("gfx950.s"))
            with open(os.path.join(temps, asm)) as fh:
                faults = check_kernels(fh.read())
            if faults:
                raise RuntimeError("%s: kernels that must not run:\n%s" % (src, "\n".join(faults[:20])))
            shutil.move(os.path.join(temps, "source.o"), obj)
        if verbose and res.stderr.strip():
            print(res.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=4) as ex:
        binding = ex.submit(_build_binding)
        objs = list(ex.map(compile_one, SOURCES))
    res = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs],
                         capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (res.stdout, res.stderr))
    binding.result()
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
