"""The host self-check of the pencil layouts refuses layouts whose rows read
their dependencies out of order or one of them twice (a small program around
the host sources plants the faults), and a layout counts as fitting only with the
LDS that its kernels hold besides the launch's."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1703_01325_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "bilu.h"
#include "bilu_internal.h"
using namespace bilu;
namespace bilu {
int device_analysis(int, const int32_t*, const int32_t*, int, int, std::vector<int32_t>&, std::vector<int32_t>&,
                    std::vector<int32_t>&, std::vector<int32_t> (&)[4]) { return BILU_ERR_ARG; }
}
// word holding dependency k of row slot q of chunk c, and its 16 bits
static int get(const HostPencil& s, int c, int q, int k)
{
    const int w4 = pencil_meta_quads(s.width), w = k / 2;
    const uint32_t two = s.meta[((static_cast<size_t>(c) * w4 + w / 4) * s.rpc + q) * 4 + w % 4];
    return k % 2 ? two >> 16 : two & 0xffffu;
}
static void set(HostPencil& s, int c, int q, int k, int code)
{
    const int w4 = pencil_meta_quads(s.width), w = k / 2;
    int32_t& two = s.meta[((static_cast<size_t>(c) * w4 + w / 4) * s.rpc + q) * 4 + w % 4];
    const uint32_t old = two;
    two = static_cast<int32_t>(k % 2 ? (old & 0xffffu) | static_cast<uint32_t>(code) << 16
                                     : (old & 0xffff0000u) | static_cast<uint32_t>(code));
}
int main(int argc, char** argv)
{
    const int nx = atoi(argv[1]), ny = atoi(argv[2]), nz = atoi(argv[3]), bs = atoi(argv[4]), k = atoi(argv[5]);
    std::vector<int32_t> Ap(1, 0), Aj;
    for (int z = 0; z < nz; ++z)
        for (int y = 0; y < ny; ++y)
            for (int x = 0; x < nx; ++x) {
                const int i = x + nx * (y + ny * z);
                if (z > 0) Aj.push_back(i - nx * ny);
                if (y > 0) Aj.push_back(i - nx);
                if (x > 0) Aj.push_back(i - 1);
                Aj.push_back(i);
                if (x + 1 < nx) Aj.push_back(i + 1);
                if (y + 1 < ny) Aj.push_back(i + nx);
                if (z + 1 < nz) Aj.push_back(i + nx * ny);
                Ap.push_back(static_cast<int32_t>(Aj.size()));
            }
    Host h;
    if (analyze_host(h, nx * ny * nz, bs, Ap.data(), Aj.data(), k, BILU_WANT_TRANSPOSE) != BILU_OK) return 2;
    int planted = 0;
    for (int w = 0; w < 4; ++w) {
        HostPencil s;
        build_pencil(h, w, h.rpc, s);
        if (!s.built || validate_pencil(h, s) != BILU_OK) return 3;
        // the LDS of a launch and the kernels' own, to the byte
        for (int cb : {1, 2}) {
            const int64_t all = pencil_lds_bytes(s.ring, s.ext_ring, s.rpc, bs, cb) + (64 + 5) * 4;
            if (!pencil_fits(s, bs, cb, all) || pencil_fits(s, bs, cb, all - 1)) return 6;
        }
        for (int c = 0; c < s.nchunks; ++c)
            for (int q = 0; q < s.rpc; ++q) {
                const size_t a = static_cast<size_t>(c) * s.width * s.rpc + q, b = a + s.rpc;
                if (s.src[a] < 0 || s.src[b] < 0) continue;     // two dependencies at least
                HostPencil bad = s;
                set(bad, c, q, 0, get(s, c, q, 1));
                set(bad, c, q, 1, get(s, c, q, 0));
                std::swap(bad.src[a], bad.src[b]);
                if (validate_pencil(h, bad) != BILU_ERR_STATE) return 4;
                bad = s;
                set(bad, c, q, 1, get(s, c, q, 0));
                bad.src[b] = bad.src[a];
                if (validate_pencil(h, bad) != BILU_ERR_STATE) return 5;
                ++planted;
            }
    }
    printf("%d\n", planted);
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    from paper_1703_01325_amd.build import CXX_FLAGS
    d = tmp_path_factory.mktemp("pencil_check")
    src = d / "driver.cpp"
    src.write_text(DRIVER)
    exe = d / "driver"
    subprocess.run(["g++", *CXX_FLAGS, "-O1", str(src), os.path.join(CSRC, "analysis.cpp"),
                    os.path.join(CSRC, "pencil.cpp"), "-o", str(exe)], check=True)
    return str(exe)


@pytest.mark.parametrize("args", [(5, 6, 4, 3, 0), (4, 5, 3, 8, 1), (3, 7, 5, 2, 2)],
                         ids=["b3k0", "b8k1", "b2k2"])
def test_self_check_refuses_disorder_and_repeats(driver, args):
    r = subprocess.run([driver, *map(str, args)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.returncode     # 3: not built, 4: swapped slots pass, 5: a repeated slot passes, 6: LDS
    assert int(r.stdout) > 100
