"""The divisions that find a work-group's tile (ks_common.hpp, Divisor): a multiplication and a shift for n / d, exact for every
n < 2^31.  The program below compares it with the division at both sides of multiples of d, for divisors around powers of two, small
ones and drawn ones."""
import os
import shutil
import subprocess

import pytest

from paper_2003_06795_amd import build as lib_build

PROGRAM = """
#include "ks_common.hpp"
#include <stdio.h>
int main() {
    unsigned long long bad = 0, seen = 0, seed = 12345;
    auto drawn = [&]() { return (unsigned)((seed = seed * 6364136223846793005ULL + 1442695040888963407ULL) >> 33); };
    auto check = [&](unsigned d) {
        if (d == 0 || d > 1u << 31) return;
        const ks::Divisor v = ks::divisor_of(d);
        auto one = [&](unsigned long long n) {
            if (n >= 1ULL << 31) return;
            ++seen;
            bad += ks::divide((unsigned)n, v) != (unsigned)n / d;
        };
        const unsigned long long top = (1ULL << 31) - 1, last = top / d * d;
        for (unsigned long long m : {0ULL, (unsigned long long)d, 2ULL * d, top / d / 2 * d, last - (last ? d : 0), last, top})
            for (int o = -1; o <= 1; ++o)
                if (o >= 0 || m > 0) one(m + o);
        for (int i = 0; i < 8; ++i) one(drawn() & 0x7FFFFFFFu);
    };
    for (unsigned d = 1; d <= 4096; ++d) check(d);
    for (int b = 12; b <= 31; ++b)
        for (int o = -3; o <= 3; ++o) check((1u << b) + o);
    for (int i = 0; i < 20000; ++i) check((drawn() & 0x7FFFFFFFu) >> (drawn() % 31));
    printf("%llu of %llu\\n", bad, seen);
    return bad != 0 || seen == 0;
}
"""


@pytest.mark.skipif(shutil.which(lib_build.HIPCC) is None, reason="needs hipcc")
def test_quotients(tmp_path):
    source, program = tmp_path / "quotients.hip", tmp_path / "quotients"
    source.write_text(PROGRAM)
    subprocess.run([lib_build.HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-I", lib_build.CSRC, str(source), "-o", str(program)],
                   check=True, capture_output=True, env=dict(os.environ))
    done = subprocess.run([str(program)], capture_output=True, text=True)
    assert done.returncode == 0, done.stdout + done.stderr
