"""The library's size rules (which launches share out their last round, which
attention kernel takes a shape), called on the host: a shim compiled against
the internal launcher header and linked to the built library.  Needs no GPU."""
import ctypes as C
import os
import subprocess

from paper_2608_09231_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
N_CU = 256
W = N_CU // 8          # work-groups per XCD of the list attention kernel
KT, QB = 64, 256       # its keys per tile and queries per item
SHARE_MIN, SPLIT_MIN = 4, 8

_SHIM = r"""
#include "paper_2608_09231_amd/csrc/kernels.h"
extern "C" {
// n problems of (M, N, K); the other arguments hold for each
int gemm_shares(int n, const int* mnk, int flags, int rms, int gelu_from, int gap_at, int gap, int gseg,
                int one_chain) {
  dit::GemmArgs g[2] = {};
  for (int i = 0; i < n; ++i) {
    const int M = mnk[3 * i], N = mnk[3 * i + 1], K = mnk[3 * i + 2];
    g[i].lda = g[i].ldw = K;
    g[i].M = M; g[i].N = N; g[i].K = K;
    g[i].ldc = N + gap;
    g[i].flags = flags; g[i].rms_cols = rms; g[i].gelu_from = gelu_from; g[i].gap_at = gap_at; g[i].gap = gap;
    g[i].gseg = gseg ? M / gseg : 0;
    g[i].one_chain = one_chain;
  }
  return dit::gemm_bf16_uses_ws(g, n, 256);
}
int attention_shares(int Lq, int Lk, int heads, int nseq) {
  return dit::flash_attn_uses_ws(Lq, Lk, heads, nseq, 256);
}
int attention_small(int Lq, int Lk, int heads, int nseq) {
  return dit::flash_attn_small_fits(Lq, Lk, heads, nseq, 256);
}
}
"""


def build(folder):
    src, out = os.path.join(folder, "plans.cpp"), os.path.join(folder, "plans.so")
    with open(src, "w") as f:
        f.write(_SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", ROOT, src, binding.LIB_PATH, "-Wl,-rpath," + os.path.dirname(binding.LIB_PATH), "-o", out],
                   check=True, capture_output=True, text=True)
    return C.CDLL(out)


def gemm_shares(lib, problems, flags=0, rms=0, gelu_from=0x7fffffff, gap_at=0x7fffffff, gap=0, gseg=0,
                one_chain=0):
    """gseg: row segments per problem with a gate vector of their own, or 0."""
    flat = [v for p in problems for v in p]
    return bool(lib.gemm_shares(len(problems), (C.c_int * len(flat))(*flat), flags, rms, gelu_from, gap_at, gap, gseg,
                                one_chain))


class AttentionPlan:
    """The list kernel's plan of one launch, per XCD 0 (the one with most
    items): whole rounds, items left over, shares of their key tiles."""

    def __init__(self, Lq, Lk, heads, nseq=1):
        items = nseq * heads * -(-Lq // QB)
        self.ntiles = -(-Lk // KT)
        self.full, self.rem = divmod(-(-items // 8), W)
        units = self.rem * self.ntiles
        self.n = max(min(units // SHARE_MIN, W), self.rem)
        self.shares = bool(self.rem) and self.ntiles - -(-units // self.n) >= SPLIT_MIN
        cuts = [units * j // self.n for j in range(self.n + 1)] if self.rem else []
        #: shares that hold parts of two items
        self.straddling = sum(a // self.ntiles != (b - 1) // self.ntiles for a, b in zip(cuts, cuts[1:]))
