"""The quotients of the KV append (csrc/tm_attn.hip): a product with a reciprocal and one correction (Markstein) are the division's
value.  The function and the refinement of the reciprocal are taken from the source and compiled for the host.

Every operand and quotient is a normal fp32 number (differences and values of fp16 numbers: 2^-24 ... 2^17), so a power of two in either
operand moves the exponent of every intermediate and no rounding: the mantissas are all there is to check, and they are checked all - 1024
by 1024 for a value over a scale, 2^23 for a range over 15 and 255.  The hardware's reciprocal is within an ulp: tried exact and an ulp
either way."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = r"""
#include <cmath>
#include <cstdio>
#include <initializer_list>
QUOTIENT
static float refined(float s, float r) { return REFINED; }
int main()
{
    long wrong = 0, checked = 0;
    for (int b = 1024; b < 2048; ++b) {
        const float s = (float)b, near = 1.0f / s;
        for (float r : {std::nextafterf(near, 0.0f), near, std::nextafterf(near, 1.0f)}) {
            const float inv = refined(s, r);
            wrong += inv != near;
            for (int a = 1024; a < 2048; ++a, ++checked) wrong += quotient((float)a, s, inv) != (float)a / s || quotient((float)-a, s, inv) != (float)-a / s;
        }
    }
    for (float top : {15.0f, 255.0f})
        for (int m = 1 << 23; m < 1 << 24; ++m, ++checked) wrong += quotient((float)m, top, 1.0f / top) != (float)m / top;
    std::printf("%ld of %ld\n", wrong, checked);
    return wrong != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_quotient_is_the_division(tmp_path):
    text = open(os.path.join(ROOT, "paper_2508_15601_amd", "csrc", "tm_attn.hip")).read()
    quotient = re.search(r"__device__ __forceinline__ (float quotient\(.*?\n}\n)", text, re.S).group(1)
    refined = re.search(r"\binv = (__builtin_fmaf\(.*\));", text).group(1)
    src, exe = tmp_path / "quotient.cpp", tmp_path / "quotient"
    src.write_text(MAIN.replace("QUOTIENT", "static " + quotient).replace("REFINED", refined))
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert done.returncode == 0 and done.stdout.strip() == f"0 of {3 * 1024 * 1024 + 2 * (1 << 23)}", done.stdout
