"""Build libqsim.so (HIP for gfx950) in-tree with hipcc.

Every .hip file under csrc/ is compiled to an object in parallel, then linked
into paper_2311_01512_amd/libqsim.so.  The headers that the specialised
tile-step kernels include are embedded in the library (they are compiled at
run time by the ROCm clang).  Packed-FP32 instructions are disabled
for all device code.
"""
import concurrent.futures as cf
import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libqsim.so")
ARCH = os.environ.get("QS_OFFLOAD_ARCH", "gfx950")

ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
HIPCC = os.environ.get("HIPCC", os.path.join(ROCM, "bin", "hipcc"))
FLAGS = ["-std=c++17", "-O3", "-fPIC", f"--offload-arch={ARCH}",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-result", "-Wno-unused-command-line-argument",
         "-I", os.path.join(HERE, "..", "include")]


# The generic kernels of tile steps and batches choose an operator by a switch
# that a whole wavefront takes alike, Pauli sums by tiles a term's pairing.  By default the compiler turns such
# branches into the chains of flags that diverging lanes need (every operator
# then passes a dozen blocks spread over 50 KiB of code, and its registers live
# across all of them); this leaves uniform regions as they are.  200 operators
# on 18 qubits in complex128 263 -> 247 us, 60 on 26 qubits in complex64
# 1974 -> 1893 us; 24 circuits of 9-14 qubits with gradients 316 -> 262 us
# (complex128 325 -> 266); 20 terms on 28 qubits 1330 -> 1270 us.
FILE_FLAGS = {f: ["-mllvm", "-structurizecfg-skip-uniform-regions"] for f in ("tiles.hip", "batch.hip", "reduce.hip")}

RTC_HEADERS = ["dev_core.hpp", "tile_dev.hpp", "batch_dev.hpp"]   # device code compiled again at run time


def _write_rtc_headers():
    """Embeds the headers the run-time compiler needs as string literals."""
    lines = ["// generated by build.py from " + ", ".join(RTC_HEADERS)]
    srcs = []
    for h in RTC_HEADERS:
        text = open(os.path.join(CSRC, h)).read()
        if ")QSRTC\"" in text:
            raise RuntimeError(f"{h} contains the raw-string delimiter")
        srcs.append('R"QSRTC(' + text + ')QSRTC"')
    lines.append(f"static const int kRtcNumHeaders = {len(RTC_HEADERS)};")
    lines.append("static const char *kRtcHeaderNames[] = {" + ", ".join(f'"{h}"' for h in RTC_HEADERS) + "};")
    lines.append("static const char *kRtcHeaderSources[] = {" + ",\n".join(srcs) + "};")
    out = os.path.join(BUILD, "qs_rtc_headers.inc")
    text = "\n".join(lines) + "\n"
    if not os.path.exists(out) or open(out).read() != text:
        open(out, "w").write(text)


# Host code built with AddressSanitizer and UndefinedBehaviorSanitizer (the
# device code is unchanged) for the CPU tests of the host logic:
# libqsim_asan.so, loaded with QS_LIB pointing at it and the clang sanitizer
# runtime preloaded.
SAN_FLAGS = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
             "-Xarch_host", "-fno-sanitize-recover=undefined", "-Xarch_host", "-fno-omit-frame-pointer"]
SAN_LIB = os.path.join(HERE, "libqsim_asan.so")


def _compile(src, san=False):
    obj = os.path.join(BUILD, os.path.basename(src) + (".san.o" if san else ".o"))
    cmd = [HIPCC] + FLAGS + FILE_FLAGS.get(os.path.basename(src), []) + (SAN_FLAGS if san else []) + ["-I", BUILD, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    err = "\n".join(l for l in r.stderr.splitlines()
                    if "packed-fp32-ops" not in l and "not a recognized feature" not in l
                    and l.strip() and "warning" in l)
    return obj, err


def build(verbose=False, jobs=None, sanitize=False):
    os.makedirs(BUILD, exist_ok=True)
    _write_rtc_headers()
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    jobs = jobs or min(len(srcs), max(1, (os.cpu_count() or 4)))
    objs = []
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        for obj, err in ex.map(lambda src: _compile(src, sanitize), srcs):
            objs.append(obj)
            if verbose and err:
                print(err, file=sys.stderr)
    out = SAN_LIB if sanitize else LIB
    tmp = out + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    if sanitize:
        cmd += ["-fsanitize=address,undefined", "-shared-libsan"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, out)
    if verbose:
        print("built", out)
    return out


if __name__ == "__main__":
    build(verbose=True)
