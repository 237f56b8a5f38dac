"""The device's gated-GELU formula, taken from its header and compiled for the host with the reciprocal off by a whole unit of its last
place either way: the error over |g| that the header of the library states, and values that are no finite numbers."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
HEADER = os.path.join(os.path.dirname(HERE), "paper_2408_06995_amd", "csrc", "gemm_common.h")
PROGRAM = r"""
#include <math.h>
#include <stdio.h>
static int off;
static float reciprocal(float v)
{
    const float r = (float)(1.0 / (double)v);
    return off == 0 || v == INFINITY ? r : nextafterf(r, off > 0 ? 2.0f : 0.0f);
}
static float maximum(float a, float b) { return a != a || b != b ? NAN : a > b ? a : b; }
static float power(float v) { return (float)exp2((double)v); }
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_rcpf reciprocal
#define __builtin_amdgcn_exp2f power
#define __builtin_elementwise_maximum maximum
%s
int main()
{
    double worst = 0.0;
    for (off = -1; off <= 1; ++off)
        for (int i = -20; i <= 5; ++i)                            // binades of the magnitude, beyond where the result is 0 or g
            for (int k = 0; k < 20000; ++k)
                for (int sign = -1; sign <= 1; sign += 2) {
                    const float g = (float)sign * (float)ldexp(1.0 + k / 20000.0, i);
                    const double e = 0.5 * (double)g * erfc(-(double)g * 0.70710678118654752440);
                    const double d = fabs((double)act_gelu(g) - e) / fabs((double)g);
                    if (!(d <= worst)) worst = d;
                }
    off = 0;
    if (!(worst < 4e-7)) return printf("error %%g\n", worst), 1;
    if (act_gelu(INFINITY) != INFINITY || act_gelu(-INFINITY) != 0.0f || act_gelu(0.0f) != 0.0f || act_gelu(NAN) == act_gelu(NAN) ||
        act_gelu(3e38f) != 3e38f || act_gelu(-3e38f) != 0.0f)
        return printf("ends\n"), 1;
    return 0;
}
"""


def test_error_and_ends(tmp_path):
    with open(HEADER) as f:
        body = re.search(r"^__device__ __forceinline__ float act_gelu\(float g\)\n\{.*?^\}", f.read(), re.S | re.M).group(0)
    src, out = str(tmp_path / "gelu.cpp"), str(tmp_path / "gelu")
    with open(src, "w") as f:
        f.write(PROGRAM % body)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-Wall", src, "-o", out])
    r = subprocess.run([out], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
