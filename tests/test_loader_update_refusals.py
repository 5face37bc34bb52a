"""The loader projections refuse a pending update where their kernels would pass it by (host checks: nothing is launched)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CALLS = r"""
#include <cstdio>
#include <cstring>
#include "gemm_skinny.h"
using namespace zo2;
// operands that are nobody's, for a process that sees no device
static zo2_status call(int dtype, int M, int K, int in_order, bool update, bool head) {
    SkinnyArgs a;
    memset(&a, 0, sizeof(a));
    void* at = (void*)(uintptr_t)(1 << 20);
    a.M = M; a.N = 128; a.K = K; a.ldx = K; a.ldy = 128; a.nprob = 1; a.eps = 1e-3f; a.in_order = in_order; a.c_ptr = update ? (const float*)at : nullptr;
    a.p[0].Xp = a.p[0].Xm = at; a.p[0].theta = at; a.p[0].Yp = a.p[0].Ym = at; a.p[0].out_scale = 1.f;
    a.labels = (const int32_t*)at; a.part_max = a.part_sum = a.label_logit = (float*)at; a.part_ld = 2 * M;
    return head ? skinny_launch_ce(a, dtype, nullptr) : skinny_launch(a, dtype, at, (size_t)1 << 40, nullptr);
}
int main() {
    int bad = 0;
    auto expect = [&](bool refused, int dtype, int M, int K, int in_order, bool update, bool head) {
        const zo2_status s = call(dtype, M, K, in_order, update, head);
        if ((s == ZO2_EINVAL) != refused || s == ZO2_OK) { printf("dtype %d M %d K %d in_order %d update %d head %d: %d\n", dtype, M, K, in_order, update, head, (int)s); ++bad; }
    };
    for (int head = 0; head < 2; ++head)
        for (int M : {1, 16, 32, 33, 96, 97, 128}) {
            for (int K : {64, 2048, 1 << 22}) {
                if ((size_t)M * K >= 0xffffffffull) continue;
                const bool fits = K < 1 << 22;
                expect(!(M <= 32 && fits), ZO2_BF16, M, K, 0, true, head);
                expect(true, ZO2_F16, M, K, 0, true, head);
                expect(false, ZO2_BF16, M, K, 0, false, head);
                expect(false, ZO2_F16, M, K, 0, false, head);
                if (!head) {
                    expect(true, ZO2_BF16, M, K, 1, true, head);
                    expect(false, ZO2_BF16, M, K, 1, false, head);
                    expect(!(M <= 96 && fits), ZO2_F32, M, K, 0, true, head);
                }
            }
        }
    printf("bad %d\n", bad);
    return bad != 0;
}
"""


def test_an_update_that_no_kernel_would_apply_is_refused(tmp_path):
    from paper_2503_12668_amd import binding, build
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    binding.lib()
    src, exe = tmp_path / "calls.cpp", tmp_path / "calls"
    src.write_text(CALLS)
    subprocess.run([hipcc, "-O1", "-std=c++17", "-x", "hip", "--offload-host-only", "-I", build.CSRC, "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe),
                    "-x", "none", build.LIB, "-Wl,-rpath," + os.path.dirname(build.LIB)], check=True)
    p = subprocess.run([str(exe)], capture_output=True, text=True, env=dict(os.environ, HIP_VISIBLE_DEVICES="", ROCR_VISIBLE_DEVICES=""))
    assert p.returncode == 0, p.stdout + p.stderr
