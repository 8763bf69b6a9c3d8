"""The library's sources built for the host with the lane scheduler of tests/simt:
the solver's device code runs on the CPU in a chosen order of waves and workgroups."""
import glob
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2405_16160_amd", "csrc")
SIMT = os.path.join(HERE, "simt")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
# what the host compiler cannot take as it stands: inline assembly, the register
# bound of a kernel and the dynamically sized LDS array
REPLACE = [
    (r'__attribute__\(\(amdgpu_waves_per_eu\(\d\)\)\)', ""),
    (r'asm volatile\("s_getreg_b32[^;]*;', "v = simt::xcd();"),
    (r'asm volatile\([^;]*;', ";"),
    (r'extern __shared__ __align__\(16\) char dyn_lds\[\];', "char* const dyn_lds = simt::dynamic_lds();"),
]


def build(out_dir):
    """Build the host library, with the C++ files of tests/simt, in out_dir; returns its path."""
    src = os.path.join(out_dir, "src")
    os.makedirs(src)
    for f in glob.glob(os.path.join(CSRC, "*")):
        name = os.path.basename(f)
        if not name.endswith((".hip", ".hpp", ".cpp")) or name == "mlp.hip":
            continue
        text = open(f).read().replace('#include "../../include/', f'#include "{ROOT}/include/')
        for pat, sub in REPLACE:
            text = re.sub(pat, sub, text)
        open(os.path.join(src, name), "w").write(text)
    for f in glob.glob(os.path.join(SIMT, "*.cpp")):
        shutil.copy(f, src)
    flags = ["-O1", "-g0", "-std=c++17", "-fPIC", "-fno-strict-aliasing", "-w", "-I", SIMT, "-I", src, "-I",
             os.path.join(ROCM, "include")]
    clang = os.path.join(ROCM, "llvm", "bin", "clang++")

    def one(f):
        obj = f + ".o"
        # (reads.cpp: every load as written, also those whose value is dropped)
        opt = ["-O0"] if f.endswith("reads.cpp") else []
        subprocess.run([clang, *flags, *opt, "-x", "c++", "-c", f, "-o", obj], check=True, capture_output=True, text=True)
        return obj

    files = glob.glob(os.path.join(src, "*.hip")) + glob.glob(os.path.join(src, "*.cpp"))
    with ThreadPoolExecutor(8) as pool:
        objs = list(pool.map(one, files))
    lib = os.path.join(out_dir, "libpdhcg_host.so")
    subprocess.run([clang, "-shared", "-Wl,-Bsymbolic", "-pthread", "-o", lib, *objs], check=True)
    return lib
