"""The bulk cache write's quotients (csrc/kv_write.hip, quantise_chunk): one reciprocal per row and a
corrected product per element must be the correctly rounded division bit for bit, for every absmax
and every element no larger that fp16 has -- zeros of both signs, subnormals and rows with an infinity
among them.  The steps are restated in C (compiled without contraction) and run on the CPU."""
import subprocess

SOURCE = r"""
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>
static uint32_t bits(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
static float fp16(int h)
{
    int e = h >> 10 & 31, m = h & 1023;
    if (e == 31) return m ? NAN : INFINITY;
    return e ? ldexpf(1024 + m, e - 25) : ldexpf(m, -24);
}
static float quotient(float x, float r, float minus_r, float s)
{
    float q0 = x * r;
    float off = fmaf(q0, s, -x);
    return fmaf(off, minus_r, q0);
}
int main(void)
{
    static float tab[0x7c01];
    const float largest[2] = {448.0f, 57344.0f};
    long bad = 0, pairs = 0;
    for (int i = 0; i <= 0x7c00; ++i) tab[i] = fp16(i);
    for (int m = 0; m < 2; ++m)
        for (int a = 0; a <= 0x7c00; ++a) {
            float scale = a == 0 ? 1.0f : tab[a] / largest[m];
            float r = 1.0f / scale, s = isinf(scale) ? 0.0f : scale;
            for (int x = 0; x <= a; ++x) {
                float p = quotient(tab[x], r, -r, s), q = tab[x] / scale;
                float pn = quotient(-tab[x], r, -r, s), qn = -tab[x] / scale;
                bad += (bits(p) != bits(q)) & !(p != p && q != q);
                bad += (bits(pn) != bits(qn)) & !(pn != pn && qn != qn);
            }
            pairs += 2 * (a + 1);
        }
    printf("%ld %ld\n", pairs, bad);
    return 0;
}
"""


def test_corrected_reciprocal_is_division(tmp_path):
    src, exe = tmp_path / "quotient.c", tmp_path / "quotient"
    src.write_text(SOURCE)
    subprocess.run(["gcc", "-O3", "-march=native", "-ffp-contract=off", str(src), "-o", str(exe), "-lm"],
                   check=True)
    pairs, bad = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert pairs == 2 * 0x7c01 * 0x7c02 and bad == 0, f"{bad} of {pairs} quotients differ"
