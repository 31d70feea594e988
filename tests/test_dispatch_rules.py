"""Which kernel takes which GEMM: the library's own predicates, called from a small host program (no GPU)."""
import os
import subprocess

import pytest

import paper_2409_15520_amd as M
from paper_2409_15520_amd import build

PROGRAM = r"""
#include "common.h"
#include "../../include/mpz.h"
#include <cstdio>
using namespace mpz;
static MfmaGemmArgs gemm(int m, int n, int k) {
  MfmaGemmArgs a{};
  a.M = m; a.N = n; a.K = k; a.w_rows = n; a.ldo = n; a.act = -1; a.rows_per_copy = m;
  return a;
}
static MfmaGemmArgs head(int m) {                        // cross-entropy partials instead of an output
  MfmaGemmArgs a = gemm(m, 50272, 2048);
  a.out_f32 = 1;
  a.ce_max = (float*)16; a.ce_sum = (float*)16; a.ce_tlogit = (float*)16; a.ce_target = (const int32_t*)16;
  return a;
}
static MfmaGemmArgs adapted(int copies, int rows) {
  MfmaGemmArgs a = gemm(copies * rows, 6144, 2048);
  a.rows_per_copy = rows; a.n_seg = 1; a.seg[0].col_begin = 0; a.seg[0].col_end = 2048; a.seg[0].rp = 32;
  return a;
}
static void say(const char* what, bool v) { printf("%s %d\n", what, (int)v); }
int main() {
  MfmaGemmArgs a = head(4096);
  say("ce", gemm_pipe_supported(a) && mfma_gemm_supported(a));
  a = head(4096); a.bias = (const float*)16; say("ce_bias", gemm_pipe_supported(a));
  a = head(4096); a.act = MPZ_ACT_RELU; say("ce_relu", gemm_pipe_supported(a));
  a = head(4096); a.n_seg = 1; a.seg[0].col_end = 2048; a.seg[0].rp = 32; say("ce_low_rank", gemm_pipe_supported(a));
  say("whole_copies", mfma_gemm_supported(adapted(8, 64)));
  say("odd_copies", mfma_gemm_supported(adapted(8, 77)) || mfma_gemm_supported(adapted(32, 77)));
  return 0;
}
"""


@pytest.fixture(scope="module")
def answers(tmp_path_factory):
    M.load_library()
    d = tmp_path_factory.mktemp("rules")
    src, obj, exe = d / "rules.hip", d / "rules.o", d / "rules"
    src.write_text(PROGRAM)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    rocm = os.path.join(os.path.dirname(os.path.realpath(hipcc)), "..", "lib")
    subprocess.run([hipcc, "--offload-host-only", "-O0", "-fPIC", "-std=c++17", "-I", build.CSRC, "-c", str(src), "-o", str(obj)], check=True,
                   capture_output=True)
    subprocess.run(["g++", str(obj), "-o", str(exe), build.LIB, "-L", rocm, "-lamdhip64", f"-Wl,-rpath,{build.PKG}", f"-Wl,-rpath,{rocm}"],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    return {l.split()[0]: l.split()[1] == "1" for l in out.splitlines()}


def test_the_cross_entropy_form_of_the_large_kernel_has_nothing_in_front_of_its_logits(answers):
    assert answers["ce"]
    assert not answers["ce_bias"] and not answers["ce_relu"] and not answers["ce_low_rank"]


def test_low_rank_terms_need_whole_copies(answers):
    assert answers["whole_copies"] and not answers["odd_copies"]
