"""The quotient of the rejection walk (csrc/quotient.h), compiled for the host, against the division it stands for: bit for bit
wherever its own conditions say that it may be used, over every exponent of dividend and divisor, subnormals among them, and
those conditions hold for what ordinary distributions bring."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include "quotient.h"
#include <stdio.h>
#include <stdint.h>
using namespace poss;
static uint64_t state = 88172645463325252ull;
static uint32_t bits() { state ^= state << 13; state ^= state >> 7; state ^= state << 17; return (uint32_t)(state >> 32); }
static float with_exponent(int e) { return ldexpf(1.f + (float)(bits() >> 9) / 8388608.f, e); }
static bool usable(float x, float z) { return quotient_divisor(z) && quotient_key(x) >= QUOTIENT_LEAST; }
static long wrong = 0, used = 0;
static void check(float x, float z) {
    if (!usable(x, z)) return;
    const volatile float d = x / z;
    const float want = d, got = quotient(x, z, 1.0f / z);
    ++used;
    if (memcmp(&want, &got, 4) && wrong++ < 5) printf("%a / %a: %a, not %a\n", x, z, got, want);
}
int main() {
    for (int ez = -149; ez <= 30; ++ez)
        for (int ex = -149; ex <= 2; ++ex)
            for (int i = 0; i < 200; ++i) check(with_exponent(ex), with_exponent(ez));
    for (int ez = -149; ez <= 30; ++ez) { check(0.f, with_exponent(ez)); check(0x1p-100f, with_exponent(ez)); }
    for (int i = 0; i < 2000000; ++i) check(with_exponent(-(int)(bits() % 60)), with_exponent((int)(bits() % 18)));
    // masses up to 1, zero among them, over totals of 1 to the vocabulary, and a residual's 1e-9: always by the quotient
    bool ordinary = usable(0.f, 1.f) && usable(1.f, 131072.f) && usable(1e-30f, 1.f) && usable(1e-9f, 1e-9f);
    bool odd = usable(1e-31f, 1.f) || usable(1e-40f, 1.f) || usable(1.f, 0.f) || usable(1.f, -1.f) || usable(1.f, 1e-39f) || usable(1.f, NAN);
    printf("used %ld wrong %ld ordinary %d odd %d\n", used, wrong, (int)ordinary, (int)odd);
    return wrong || !ordinary || odd;
}
"""


def test_quotient_is_the_division_wherever_it_is_used(tmp_path):
    src, exe = tmp_path / "quotient.cc", tmp_path / "quotient"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-I", os.path.join(ROOT, "paper_2506_03566_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    print(r.stdout)
    assert r.returncode == 0
