"""Operands of the kernels' inline assembly, from the compiler's own listing for gfx950 (no GPU needed).

A statement of several instructions writes its accumulators before it has read all of its inputs.  Without an early clobber the compiler may
give an input the register of an accumulator that has the same value on entry; the calls here have such values."""
import os
import re
import subprocess

import pytest

from paper_2502_07861_amd.build import CSRC, FLAGS

SOURCE = r"""
#include "bkv_device.h"
#include "walk_quarters.h"
using namespace bkv;
template <int N> __global__ void dot_kernel(const float* in, float* out) {
    float f[N];
    for (int i = 0; i < N; ++i) f[i] = in[64 * i + threadIdx.x];
    float acc = f[N - 1];
    dpp_dot<0>(acc, in[64 * N + threadIdx.x], f);
    out[threadIdx.x] = acc;
}
template __global__ void dot_kernel<4>(const float*, float*);
template __global__ void dot_kernel<8>(const float*, float*);
template <int B> __global__ void steps_kernel(const float* in, float* out, unsigned int sign_bit) {
    float g[64];
    for (int i = 0; i < 64; ++i) g[i] = i >= B && i < B + 8 ? in[64 * i + threadIdx.x] : 0.f;
    float s = g[B + 6];
    walk_steps8<B>(s, g, sign_bit);
    out[threadIdx.x] = s;
}
template __global__ void steps_kernel<8>(const float*, float*, unsigned int);
template __global__ void steps_kernel<40>(const float*, float*, unsigned int);
template <int WHICH> __global__ void walk_kernel(const float* in, float* out, unsigned int m) {
    float c[16], a[16], b[16];
    for (int i = 0; i < 16; ++i) { c[i] = in[64 * i + threadIdx.x]; a[i] = in[64 * (16 + i) + threadIdx.x]; b[i] = in[64 * (32 + i) + threadIdx.x]; }
    float s = c[6], p = a[5], q = b[6], z = in[64 * 48 + threadIdx.x];
    if constexpr (WHICH == 0) z = walk_both<0>(s, p, q, c, a, b, m);
    else if constexpr (WHICH == 1) z = walk_mix<0>(s, p, q, z, c, a, b, m);
    else if constexpr (WHICH == 2) { q = a[13]; walk_late<0>(s, q, z, c, a, m); }
    else walk_plain<0>(s, c, m);
    out[threadIdx.x] = s; out[64 + threadIdx.x] = p; out[128 + threadIdx.x] = q; out[192 + threadIdx.x] = z;
}
template __global__ void walk_kernel<0>(const float*, float*, unsigned int);
template __global__ void walk_kernel<1>(const float*, float*, unsigned int);
template __global__ void walk_kernel<2>(const float*, float*, unsigned int);
template __global__ void walk_kernel<3>(const float*, float*, unsigned int);
"""


def test_accumulators_share_no_register_with_inputs(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no compiler")
    src, out = tmp_path / "operands.hip", tmp_path / "operands.s"
    src.write_text(SOURCE)
    subprocess.run([hipcc, *FLAGS, "-I" + CSRC, "--offload-device-only", "-S", str(src), "-o", str(out)], check=True, capture_output=True)
    statements = [s for pair in re.findall(r";\s?APP\n(.*?);\s?NO_APP|#ASMSTART\n(.*?)#ASMEND", out.read_text(), re.S) for s in pair if s.count("v_fmac_f32") >= 4]
    assert len(statements) == 8
    for s in statements:
        adds = re.findall(r"v_fmac_f32(?:_dpp)? (v\d+), -?(v\d+), (v\d+)", s)
        assert len(adds) >= 4
        written = {d for d, _, _ in adds}
        assert not written & {g for _, _, g in adds}, s
