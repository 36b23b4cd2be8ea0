"""A CPU build of the library's kernels, for the tests: every lane a fibre, every access checked (lanes.cpp).

The sources are taken as they are but for pointers with an address space, which become objects that check what they point
at, and two instructions that are written in assembly.  The matrix-core kernel, whose loop is in assembly, is left out; the dispatch for it and
the copy of activations into its blocks, which a layer call without it does not reach, have entries here.
"""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_2310_16795_amd", "csrc")
UNITS = ["qmoe_host.cpp", "qmoe_api.hip", "qmoe_product_sym.hip", "qmoe_product_asym.hip", "qmoe_rows.hip", "qmoe_dispatch.hip", "qmoe_matvec.hip",
         "qmoe_decompress.hip", "qmoe_encode.hip", "qmoe_misc.hip"]
NO_MATRIX_CORES = """#include "qmoe_dev.h"
namespace qmoe {
size_t mm_lds_bytes(int) { return (size_t)1 << 40; }
qmoe_status launch_product_mm(ProductArgs, const MmPlan &, hipStream_t) { return QMOE_E_LIMIT; }
}
using namespace qmoe;
extern "C" int lanes_tile_x(const int *items, const int *n_items, int max_items, const int *perm, const uint16_t *x, int cols, uint16_t *out, int cus)
{
    ProductArgs a{};
    a.items = reinterpret_cast<const Item *>(items);
    a.n_items_dev = n_items;
    a.max_items = max_items;
    a.perm = perm;
    a.x = x;
    a.cols = a.ldx = cols;
    return launch_tile_x(a, out, cus, nullptr);
}
extern "C" int lanes_dispatch(const int32_t *expert_idx, int n_tokens, int n_experts, int *tok_off, int *perm, int *counters, int *items_wi, int *items_wo,
                              int *items_mm, const int *lines /*mm_min, mm_from, mm_else, mm_below, mm_passes, mm_split*/, float *y, int d_model, int max_lds)
{
    auto list = [](int *p) { return reinterpret_cast<Item *>(p); };
    const DispatchArgs d{expert_idx, n_tokens, n_experts, tok_off, perm, counters, list(items_wi), list(items_wo), list(items_mm), 4, 4,
                         lines[0], lines[1], lines[2], lines[3], lines[4], lines[5], y, d_model};
    return launch_dispatch_kernel(d, max_lds, nullptr);
}
"""


def converted(text: str) -> str:
    space = r"__attribute__\(\(address_space\((\d)\)\)\) "
    text = re.sub("typedef const " + space + r"([\w ]+?) \*(\w+);", r"typedef lanes::Ptr<\1, const \2> \3;", text)
    text = re.sub("typedef " + space + r"([\w ]+?) \*(\w+);", r"typedef lanes::Ptr<\1, \2> \3;", text)
    text = re.sub("const " + space + r"(unsigned long long|unsigned char|\w+) \*", r"lanes::Ptr<\1, const \2> ", text)
    text = re.sub(space + r"(unsigned long long|unsigned char|\w+) \*", r"lanes::Ptr<\1, \2> ", text)
    text = text.replace("extern __shared__ __align__(16) unsigned char smem[];", "unsigned char *smem = lanes::lds();")
    text = text.replace("extern __shared__ int sm[];", "int *sm = reinterpret_cast<int *>(lanes::lds());")
    text = text.replace("tile.tok_ids = g->tok;", "tile.tok_ids = lanes::Ptr<3, const int>(&g->tok[0]);")
    text = text.replace('asm("v_lshl_or_b32 %0, %1, 25, %2" : "=v"(f) : "v"(two), "v"(two << 18));', "f = (two << 25) | (two << 18);")
    text = re.sub(r'asm\("v_med3_u32 %0, %1, %2, %3" : "=v"\((\w+)\) : "v"\((.*?)\), "v"\((\w+)\), "s"\(last\)\);', r"\1 = lanes_med3(\2, \3, last);", text)
    return text


def build(into: str) -> str:
    src = os.path.join(into, "src")
    os.makedirs(src, exist_ok=True)
    for name in os.listdir(CSRC):
        if name.endswith((".h", ".hip", ".cpp")):
            with open(os.path.join(CSRC, name)) as f, open(os.path.join(src, name), "w") as g:
                g.write(converted(f.read()))
    with open(os.path.join(src, "no_matrix_cores.cpp"), "w") as f:
        f.write(NO_MATRIX_CORES)
    files = [os.path.join(src, u) for u in UNITS + ["no_matrix_cores.cpp"]] + [os.path.join(HERE, "lanes.cpp")]
    clang = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")
    jobs = [(f, subprocess.Popen([clang, "-x", "c++", "-O1", "-std=c++17", "-fPIC", "-w", "-I", HERE, "-I", src, "-I", os.path.join(ROOT, "include"),
                                  "-c", f, "-o", os.path.join(into, os.path.basename(f) + ".o")], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
            for f in files]
    for f, p in jobs:
        out = p.communicate()[0]
        assert p.returncode == 0, f"{f}\n{out[-3000:]}"
    lib = os.path.join(into, "libqmoe_lanes.so")
    subprocess.check_call([clang, "-shared", "-o", lib, *[os.path.join(into, os.path.basename(f) + ".o") for f in files], "-lpthread"])
    return lib
