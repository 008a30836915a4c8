"""Compiles the library's sources for the CPU, against the HIP of hip/hip_runtime.h, into a library with the same C ABI."""
import glob
import os
import re
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_2207_11019_amd", "csrc")

# global memory straight to LDS: the same calls without the GPU's assembly
LDS_DMA = """#pragma once
#include <hip/hip_runtime.h>
namespace lpm {
#define LPM_WAIT_VM(n) lanes::wait_loads(n)
typedef unsigned int u32x4_ __attribute__((ext_vector_type(4)));
inline u32x4_ buffer_words(const void* base, unsigned bytes) {
    const unsigned long long a = (unsigned long long)base;
    const u32x4_ r = {(unsigned)a, (unsigned)(a >> 32) & 0xffffu, bytes, 0x00020000u};
    return r;
}
inline void load_to_lds16s(u32x4_ rs, const unsigned char* dst, unsigned off, unsigned soff) {
    const unsigned w[4] = {rs.x, rs.y, rs.z, rs.w};
    lanes::load_to_lds(w, (unsigned char*)dst, off, (unsigned)__builtin_amdgcn_readfirstlane((int)soff));
}
inline void load_to_lds16(u32x4_ rs, const unsigned char* dst, unsigned off) {
    const unsigned w[4] = {rs.x, rs.y, rs.z, rs.w};
    lanes::load_to_lds(w, (unsigned char*)dst, off, 0);
}
}
"""
# the LDS transpose read: lane i of 16 receives element i % 4 of the rows that lanes 4j + i/4 point at
TR4 = """inline u32x2_ tr4(const unsigned char* p) {
    const unsigned char* x = lanes::exchange(&p, sizeof p, __LINE__);
    unsigned short e[4];
    const int g = lanes::lane & ~15, i = lanes::lane & 15;
    for (int j = 0; j < 4; ++j) {
        const unsigned char* q;
        memcpy(&q, x + (size_t)(g + 4 * j + i / 4) * sizeof p, sizeof p);
        memcpy(&e[j], q + 2 * (i % 4), 2);
    }
    (void)lane_value(0, 0, __LINE__);
    u32x2_ r = {(unsigned)e[0] | ((unsigned)e[1] << 16), (unsigned)e[2] | ((unsigned)e[3] << 16)};
    return r;
}
"""


def _host_form(name, t):
    if name == "lds_dma.h":
        return LDS_DMA
    t = t.replace('"../../include/lpm.h"', '"lpm.h"')
    t = re.sub(r"extern __shared__ (?:__attribute__\(\(aligned\(16\)\)\) )?(unsigned char|float) (\w+)\[\];", r"\1* \2 = (\1*)lanes::dynamic_lds();", t)
    t = t.replace('asm volatile("s_waitcnt vmcnt(0)" ::: "memory");', "lanes::wait_loads(0);")
    t = t.replace("& 255u", "& 15u")           # (host tensors are aligned to 64 bytes)
    if name == "elem.h":            # the element-by-element loads are counted
        t, n = re.subn(r"(__device__ __forceinline__ float ld\(const \w+\* p, int64_t i\) \{) ", r"\1 ++lanes::element_loads; ", t)
        assert n == 2, "the loads of elem.h have changed their form"
    if name == "wgrad.hip":
        t, n = re.subn(r"__device__ __forceinline__ u32x2_ tr4\(.*?\n}\n", lambda m: TR4, t, flags=re.S)
        assert n == 1, "the transpose read of wgrad.hip has changed its form"
    t = re.sub(r'asm volatile\("" ?:.*?\);', "", t)
    assert "asm" not in re.sub(r"//.*", "", t), name + " holds assembly that this build does not know"
    return t


def build(out, flags=(), extra=(), exe=None, opt="-O2"):
    """liblanes.so (or, with exe, a program of the sources in `extra`) in directory `out`; returns its path."""
    src = os.path.join(out, "src")
    os.makedirs(src, exist_ok=True)
    for p in glob.glob(os.path.join(CSRC, "*")):
        with open(p) as f, open(os.path.join(src, os.path.basename(p)), "w") as o:
            o.write(_host_form(os.path.basename(p), f.read()))
    shutil.copy(os.path.join(ROOT, "include", "lpm.h"), src)
    cxx = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")
    common = [cxx, "-x", "c++", "-std=c++17", opt, "-g1", "-fPIC", "-Wno-everything", "-I" + HERE, "-I" + src, *flags]
    procs, objs = [], []
    for p in [os.path.join(HERE, "lanes.cpp"), os.path.join(HERE, "routes.cpp"), *extra] + sorted(glob.glob(os.path.join(src, "*.hip")) + glob.glob(os.path.join(src, "*.cpp"))):
        o = os.path.join(out, os.path.basename(p) + ".o")
        objs.append(o)
        procs.append(subprocess.Popen(common + ["-c", p, "-o", o], stderr=subprocess.PIPE, text=True))
    for p in procs:
        _, err = p.communicate()
        assert p.returncode == 0, err[-4000:]
    target = os.path.join(out, exe or "liblanes.so")
    link = [f for f in flags if f.startswith("-fsanitize")]
    subprocess.check_call([cxx, *link, *([] if exe else ["-shared"]), "-o", target, *objs, "-lpthread", "-ldl"])
    return target
