"""The library's rules (csrc/plan.h) as ctypes functions, compiled for the host alone.  Not collected by pytest (no test_ prefix)."""
import ctypes
import os
import subprocess

from paper_2011_09208_amd import buildlib

PLAN = os.path.join(buildlib.PKG, "csrc", "plan.h")
STEP, PROBS, TOP1, FORWARD = 0, 1, 2, 3                  # SmallUse, and the forward call's own
SMALL, BLOCKS, LISTS, TILES = 0, 1, 2, 3                 # LogitsWay
SHIM = """#include "%s"
using namespace ws;
extern "C" {
size_t fwd_bytes_(int B, int D, int C) { return fwd_bytes(B, D, C); }
size_t least_fwd_bytes_(int B, int C) { return least_fwd_bytes(B, C); }
static LogitsPlan plan(int B, int D, int C, int use) {
    return use == 3 ? plan_forward(B, D, C, plan_logits(B, D, C, SMALL_STEP)) : plan_logits(B, D, C, (SmallUse)use);
}
size_t way_bytes_(int B, int D, int C, int use) { return plan(B, D, C, use).bytes(); }
int way_(int B, int D, int C, int use) { return plan(B, D, C, use).way; }
unsigned quotient_(unsigned n, unsigned d) { return quotient(n, inverse(d)); }
unsigned list_quotient_(unsigned n, int D, int C, int nBT) { return quotient(n, plan_ranges(D, C, nBT).inv_ranges); }
int descending_(int B, int D, int C, int ct, int bt) {
    const LogitsPlan p = plan_logits(B, D, C, SMALL_STEP);
    return logits_descending(logits_order(p), p.ranges, (B + 255) / 256, ct, bt);
}
int ranges_(int D, int C, int nBT) { return plan_ranges(D, C, nBT).ranges; }
void dx_splits_(int B, int D, int C, int* out) {
    const BwdPlan p = plan_bwd(B, D, C);
    out[0] = p.dx_small;
    out[1] = p.splits;
    out[2] = p.steps_per_split;
    out[3] = p.dw_small;
}
size_t bwd_bytes_(int B, int D, int C) { return plan_bwd(B, D, C).bytes(); }
}
"""


def load(folder):
    """Compiles the rules in `folder` and loads them."""
    src, lib = os.path.join(folder, "rules.hip"), os.path.join(folder, "rules.so")
    with open(src, "w") as f:
        f.write(SHIM % PLAN)
    subprocess.run([buildlib.HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wno-unused-function",
                    src, "-o", lib], check=True)
    rules = ctypes.CDLL(lib)
    for name in ("fwd_bytes_", "least_fwd_bytes_", "way_bytes_", "bwd_bytes_"):
        getattr(rules, name).restype = ctypes.c_size_t
    rules.quotient_.restype = rules.list_quotient_.restype = ctypes.c_uint
    return rules
