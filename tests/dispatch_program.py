"""The library's own dispatch rules, asked from a small host program (no GPU): ask() takes lines of a query's name and its numbers and
returns one integer per line."""
import functools
import os
import subprocess
import tempfile

import paper_2409_15520_amd as M
from paper_2409_15520_amd import build

PROGRAM = r"""
#include "common.h"
#include "../../include/mpz.h"
#include <cstdio>
#include <cstring>
using namespace mpz;
int main() {
  char what[64];
  while (scanf("%63s", what) == 1) {
    if (!strncmp(what, "lora_down_ordered", 17)) {       // K, rank, targets, rows per copy, copies
      LoraDownArgs a{};
      int copies;
      if (scanf("%d %d %d %d %d", &a.K, &a.rank, &a.n_targets, &a.rows_per_copy, &copies) != 5) return 1;
      a.dtype = MPZ_DTYPE_BF16; a.T = copies * a.rows_per_copy; a.x = (const void*)4096; a.copy_stride = 16LL * a.K * a.rank;
      for (int t = 0; t < a.n_targets; ++t) a.Ac[t] = (const float*)4096 + 2LL * t * a.K * a.rank;
      if (!strcmp(what, "lora_down_ordered_launch")) {     // did it launch?  Asked only where there is no device to launch on
        int devices = 0;
        if (hipGetDeviceCount(&devices) == hipSuccess && devices > 0) return 1;
        printf("%d\n", (int)launch_lora_down_ordered(nullptr, a));
      } else
        printf("%lld\n", (long long)lora_down_ordered_blocks(a));
    } else if (!strcmp(what, "tile")) {                  // M, N, K, bits of a weight, rotated columns (-1: gate and up), their heads: tile, or -1 if refused
      MfmaGemmArgs a{};
      int bits;
      if (scanf("%d %d %d %d %d %d", &a.M, &a.N, &a.K, &bits, &a.rope_cols, &a.rope_dh) != 6) return 1;
      a.w_rows = a.ldo = a.N; a.act = -1; a.rows_per_copy = a.M; a.x = a.w = a.out = (void*)4096;
      if (bits == 8) a.w_scale = (const float*)4096;
      if (a.rope_cols < 0) { a.rope_cols = 0; a.dual = 1; a.dual_offset = a.N; a.w_rows = 2 * a.N; }
      if (a.rope_cols) { a.rope_cos = a.rope_sin = (const float*)4096; a.S = a.M; }
      printf("%d\n", mfma_gemm_supported(a) ? mfma_gemm_tile(a) : -1);
    } else if (!strcmp(what, "nf4_run")) {               // M, N, K of 4-bit weights, rows of partial sums there is room for: K-tiles per block of the streamed kernel
      MfmaGemmArgs a{};
      long rows;
      if (scanf("%d %d %d %ld", &a.M, &a.N, &a.K, &rows) != 4) return 1;
      a.w_rows = a.N; a.x = a.w = (const void*)4096; a.w_absmax = (const float*)4096; a.rows_per_copy = a.M;
      printf("%d\n", gemm_codes_plan(a, (size_t)rows * a.N, false));
    } else if (!strcmp(what, "attention_f64")) {         // sequences, tokens, heads, columns of a head: taken?
      int n, S, H, dh;
      if (scanf("%d %d %d %d", &n, &S, &H, &dh) != 4) return 1;
      printf("%d\n", (int)attention_f64_supported((const float*)4096, 3 * H * dh, n, S, H, dh));
    } else if (!strcmp(what, "attention_keeps")) {       // sequences, tokens, heads, key-value heads, columns of a head
      int n, S, H, kv, dh;
      if (scanf("%d %d %d %d %d", &n, &S, &H, &kv, &dh) != 5) return 1;
      printf("%d\n", (int)attention_keeps_scores(n, S, H, kv, dh));
    } else if (!strcmp(what, "attention_eight")) {       // sequences, tokens, heads, columns of a head
      int n, S, H, dh;
      if (scanf("%d %d %d %d", &n, &S, &H, &dh) != 4) return 1;
      printf("%d\n", (int)attention_eight_waves(n, S, H, dh));
    } else if (!strcmp(what, "attention_far")) {         // tokens of a sequence, heads, key-value heads, columns of a head
      int S, H, kv, dh;
      if (scanf("%d %d %d %d", &S, &H, &kv, &dh) != 4) return 1;
      printf("%d\n", (int)attention_far(S, (H + 2 * kv) * dh, kv * dh));
    } else if (!strcmp(what, "two_halves")) {            // d, columns of Q|K|V, d_ffn, gate and up, weight_quant, stacked tokens
      int d, nqkv, ffn, gate, quant, T;
      if (scanf("%d %d %d %d %d %d", &d, &nqkv, &ffn, &gate, &quant, &T) != 6) return 1;
      printf("%d\n", (int)two_halves_pay(d, nqkv, ffn, gate != 0, quant, T));
    } else return 1;
  }
  return 0;
}
"""


_DIR = tempfile.TemporaryDirectory()


@functools.lru_cache(maxsize=None)
def _program():
    M.load_library()
    src, obj, exe = (os.path.join(_DIR.name, n) for n in ("rules.hip", "rules.o", "rules"))
    with open(src, "w") as f:
        f.write(PROGRAM)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    rocm = os.path.join(os.path.dirname(os.path.realpath(hipcc)), "..", "lib")
    subprocess.run([hipcc, "--offload-host-only", "-O0", "-fPIC", "-std=c++17", "-I", build.CSRC, "-c", src, "-o", obj], check=True,
                   capture_output=True)
    subprocess.run(["g++", obj, "-o", exe, build.LIB, "-L", rocm, "-lamdhip64", f"-Wl,-rpath,{build.PKG}", f"-Wl,-rpath,{rocm}"],
                   check=True, capture_output=True)
    return exe


def ask(lines):
    out = subprocess.run([_program()], input="\n".join(lines) + "\n", check=True, capture_output=True, text=True,
                         env=dict(os.environ, HIP_VISIBLE_DEVICES="-1")).stdout.split()
    assert len(out) == len(lines)
    return [int(v) for v in out]
