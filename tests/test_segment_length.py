"""Scaled lengths of the segment tables (segment_length.h), compiled for the
host: a length kept as FP32 and its rest gives the FP32 value of the FP64
product length x scale, as the walk forms it."""
import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2408_14425_amd", "csrc")

CODE = r"""
#include "segment_length.h"
#include <cmath>
#include <cstdio>
#include <random>
int main()
{
    std::mt19937_64 rng(3);
    std::uniform_real_distribution<double> u(0.0, 1.0);
    long wrong = 0, far = 0, plain = 0, n = 2000000;
    for (long i = 0; i < n; ++i) {
        const double len = i % 8 ? 1.4142135623730951 * u(rng) : std::ldexp(u(rng), -30);
        const double mu = 0.999 * u(rng), scale = 1.0 / std::sqrt(1.0 - mu * mu);
        const float want = (float)(len * scale);
        const float got = rcx::scaled_length((float)len, rcx::length_rest(len), scale);
        wrong += got != want;
        far += std::fabs(got - want) > std::ldexp(std::fabs(want), -23);
        plain += (float)len * (float)scale != want;
    }
    std::printf("%ld %ld %ld\n", wrong, far, plain);
}
"""


def test_scaled_length_rounds_once(tmp_path):
    """The rest holds 24 more bits of the length, so the product differs from
    the FP64 one by 2^-47 of it and rounds elsewhere once in 2^22 at most; the
    product of the rounded numbers is off in a large part of the cases."""
    cxx = os.environ.get("CXX") or shutil.which("g++") or "/opt/rocm/llvm/bin/clang++"
    src = tmp_path / "t.cpp"
    src.write_text(CODE)
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, "-o", str(tmp_path / "t"), str(src)], check=True)
    wrong, far, plain = map(int, subprocess.run([str(tmp_path / "t")], capture_output=True, text=True, check=True).stdout.split())
    assert wrong <= 5 and far == 0, (wrong, far)
    assert plain > 100000


def test_inclined_solvers_keep_the_rests(tmp_path):
    """The tables of a non-LTE solver with inclinations hold them."""
    from host_runtime import run
    run(tmp_path, """
        from paper_2408_14425_amd import workloads
        atm = workloads.nlte_atmosphere(64, seed=5, n_line=16, n_cont=8)
        size = []
        for n_incl in (1, 2):
            mallocs()
            h = rcx.rcx_nlte_create(rcx.rcx_grid(64, 64, 1.0), params(n_incl=n_incl), rcx.atom_from_dict(atm.atom),
                                    atm.lambda_nm, atm.trans, atm.dnu)
            size.append(mallocs()[1])  # the tables
            rcx.rcx_nlte_destroy(h)
        assert size[1] > size[0] + size[0] // 5, size
    """)
