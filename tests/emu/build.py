"""Builds the CPU emulation of libgspar (test infrastructure): the unchanged HIP source compiled
with g++ against tests/emu/hip/hip_runtime.h, optionally with AddressSanitizer."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
SRC = os.path.join(ROOT, "paper_1710_09854_amd", "csrc", "gspar.hip")
OUT_DIR = os.path.join(HERE, "_build")


def build(asan: bool = False, concurrent: bool = False) -> str:
    os.makedirs(OUT_DIR, exist_ok=True)
    res = os.environ.get("GSPAR_EMU_RESIDENT")
    # rows from this length on predict a candidate band (a small threshold and sample exercise the
    # band on the emulated sizes; the production threshold exercises refinement over the row)
    cmin = int(os.environ.get("GSPAR_EMU_CAND_MIN_ROW", "4096"))
    # keys of a range up to which the solver lists them; a small value exercises its windows and counts
    lst = os.environ.get("GSPAR_EMU_LIST")
    # helpers of the solver resident at once; a small value makes each take several chunks of a row
    hlp = os.environ.get("GSPAR_EMU_HELPERS")
    out = os.path.join(OUT_DIR, ("libgspar_emu_asan" if asan else "libgspar_emu") + (f"_r{int(res)}" if res else "")
                       + f"_c{cmin}" + (f"_l{int(lst)}" if lst else "") + (f"_h{int(hlp)}" if hlp else "")
                       + ("_conc" if concurrent else "") + ".so")
    if os.path.exists(out) and os.path.getmtime(out) > max(os.path.getmtime(SRC),
                                                         os.path.getmtime(os.path.join(HERE, "hip", "hip_runtime.h"))):
        return out
    tmp = f"{out}.{os.getpid()}.tmp"
    # a short look-back wait keeps the emulated fallback test (every status hidden) quick; a low
    # residency threshold makes the small emulated inputs take the two-tiles-per-workgroup path too
    # when GSPAR_EMU_RESIDENT is set
    # (-fno-gnu-unique: two builds loaded into one process share no inline or function-local variable)
    cmd = ["g++", "-std=c++20", "-O1", "-g", "-fPIC", "-shared", "-pthread", "-fno-gnu-unique", "-Wno-attributes",
           "-DGSPAR_LOOKBACK_POLLS=64",
           f"-DGSPAR_SAMPLE_RESIDENT={int(os.environ.get('GSPAR_EMU_RESIDENT', '1792'))}",
           f"-DGSPAR_CAND_MIN_ROW={cmin}", "-DGSPAR_PRE_LINES=64",
           "-Wno-unknown-pragmas", "-I", HERE, "-I", os.path.join(ROOT, "include"), "-x", "c++", SRC,
           "-o", tmp]
    if lst:
        cmd.insert(1, f"-DGSPAR_LIST_CAP={int(lst)}")
    if hlp:
        cmd.insert(1, f"-DGSPAR_SOLVE_HELPERS={int(hlp)}")
    if concurrent:
        cmd.insert(1, "-DEMU_CONCURRENT")
    if asan:
        cmd[1:1] = ["-fsanitize=address", "-fno-omit-frame-pointer"]
    subprocess.run(cmd, check=True)
    os.replace(tmp, out)
    return out


def asan_runtime() -> str:
    return subprocess.run(["g++", "-print-file-name=libasan.so"], capture_output=True, text=True,
                          check=True).stdout.strip()


if __name__ == "__main__":
    print(build(False), build(True))
