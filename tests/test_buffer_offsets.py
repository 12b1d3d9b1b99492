"""The 32-bit byte offsets of the staple passes' buffer accesses (csrc/su3.h).

Planes 0-4 of a field share one buffer resource of 2^32 - 1 bytes: plane 4
starts 64 P bytes into it and a lane adds up to 16 P, P the plane stride in
sites.  The range check may count the sum, so the whole of it has to fit."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1712_00143_amd", "csrc")

PROBE = r"""
#include <cstdio>
#include <cstdlib>
#include "gforce.h"
int main(int argc, char **argv)
{
    std::printf("%lld", (long long)hisq::BUF_MAX_P);
    for (int k = 1; k < argc; k++) std::printf(" %lld", hisq::plane_stride(std::atoll(argv[k])));
    std::printf("\n");
}
"""


def _probe(tmp_path, volumes):
    src, exe = tmp_path / "probe.cpp", tmp_path / "probe"
    src.write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src), "-o",
                    str(exe)], check=True, capture_output=True, text=True)
    out = subprocess.run([str(exe)] + [str(v) for v in volumes], check=True, capture_output=True, text=True).stdout
    vals = [int(x) for x in out.split()]
    return vals[0], vals[1:]


def test_last_byte_of_the_last_plane_fits_the_resource(tmp_path):
    vols = [32 ** 4, 64 ** 3 * 200, 84 ** 4, 64 ** 3 * 208, 88 ** 4, 90 ** 3 * 92]
    bound, strides = _probe(tmp_path, vols)
    records = 2 ** 32 - 1
    largest = (bound - 1) // 8 * 8          # strides are multiples of 8 below the bound
    assert 4 * 16 * largest + 16 * largest <= records
    # lattices that fit are served, 88^4 and above are not
    for v, p in zip(vols, strides):
        fits = 5 * 16 * p <= records
        assert (p < bound) == fits, (v, p)


RULE = r"""
#include <cstdio>
#include <cstdlib>
#include "gforce.h"
int main(int argc, char **argv)
{
    for (int k = 1; k < argc; k++) {
        hisq::SmearGeom g{};
        g.V = std::atoll(argv[k]);
        g.P = hisq::plane_stride(g.V);
        std::printf("%d%d ", hisq::gauge_force_even_serves(g, -0.08), hisq::gauge_force_even_serves(g, 0.0));
    }
}
"""


def test_gauge_force_kernel_rule(tmp_path):
    """Which lattices the kernel around even sites serves, with and without
    rectangles: not the small ones, nor those beyond its offsets."""
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(RULE)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src), "-o",
                    str(exe)], check=True, capture_output=True, text=True)
    vols = {8192: "00", 8208: "01", 16384: "01", 16400: "11", 32 ** 4: "11", 84 ** 4: "11", 64 ** 3 * 200: "11",
            64 ** 3 * 208: "00", 88 ** 4: "00", 100 ** 4: "00"}
    out = subprocess.run([str(exe)] + [str(v) for v in vols], check=True, capture_output=True, text=True).stdout
    assert out.split() == list(vols.values())
