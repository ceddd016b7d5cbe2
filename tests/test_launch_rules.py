"""Host-side launch rules of the kernels, compiled alone for the CPU: no GPU call is made."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0704_0037_amd", "csrc")


def _run(tmp_path, text):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "probe.hip", tmp_path / "probe"
    src.write_text(text)
    subprocess.run([hipcc, "--offload-host-only", "-O0", "-std=c++17", "-Wno-everything", "-I", CSRC, "-I",
                    os.path.join(CSRC, "..", "..", "include"), str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()


def test_lds_limit_of_a_kernel_is_never_lowered(tmp_path):
    """The column kernel's dynamic LDS follows the grid and the number of vectors (L = 256: 78,240 and
    65,856 bytes), and the limit set for a kernel is the last one set: whatever the order of the calls,
    the limit at every launch covers that launch."""
    out = _run(tmp_path, """
#include <hip/hip_runtime.h>
#include <cstdio>
static int limit = 65536;
static hipError_t set_limit(const void *, hipFuncAttribute, int v) { limit = v; return hipSuccess; }
static hipError_t device(int *d) { *d = 0; return hipSuccess; }
#define hipFuncSetAttribute set_limit
#define hipGetDevice device
#include "matvec_launch.hpp"
namespace dda { void set_error(const std::string &) {} }
static void kernel() {}
int main() {
    using namespace dda;
    auto size = [](int noct, int n) {
        const ZShape z = zcol_shape<double, 256>(noct, n);
        return zcol_lds<double, 256>(z.opb, z.W);
    };
    const size_t a = size(1285, 5), b = size(257 * 257, 9);
    for (size_t bytes : {a, b, a, b, (size_t)1024, a}) {
        allow_lds(&kernel, bytes);
        std::printf("%zu %d\\n", bytes, limit);
    }
}
""")
    pairs = [(int(out[i]), int(out[i + 1])) for i in range(0, len(out), 2)]
    assert len({b for b, _ in pairs if b > 65536}) == 2  # two sizes above the default limit
    assert all(b <= lim for b, lim in pairs), pairs


def _setup(grid, pad, mask=None):
    """Status and message of a dda_setup call that is to end before any device call."""
    import ctypes as ct

    from paper_0704_0037_amd import dda
    L = dda.lib()
    L.dda_last_error.restype = ct.c_char_p
    h = ct.c_void_p()
    cells = (ct.c_uint8 * (grid[0] * grid[1] * grid[2]))(1)
    opts = dda.SetupOpts()
    opts.pad[:] = pad
    st = L.dda_setup(ct.byref(h), (ct.c_int32 * 3)(*grid), cells, (ct.c_double * 2)(1.5, 0.0), 0.4, 0, ct.byref(opts), None)
    assert h.value is None
    return st, L.dda_last_error()


@pytest.mark.parametrize("pad", [405, 486, 540, 600, 1024, 4096])
def test_z_lines_wider_than_a_wave_are_refused(pad):
    """L / (largest radix) > 64 lanes leaves the z pass no slot for a column: refused before any device
    call (405 and 486 have no radix 8, the others are longer than 512)."""
    from paper_0704_0037_amd import dda
    st, why = _setup((2, 2, 100), (4, 4, pad))
    assert st == dda.EINVAL and b"padded size too large" in why


@pytest.mark.timeout(60, method="thread")
@pytest.mark.parametrize("nz", [257, 300, 2047, 2048])
def test_default_padding_ends_for_long_axes(nz):
    """No padded length above 512 fits the z pass: more than 256 cells along z are refused, not searched
    for without end."""
    from paper_0704_0037_amd import dda
    st, why = _setup((2, 3, nz), (0, 0, 0))
    assert st == dda.EINVAL and b"padded size too large" in why


@pytest.mark.timeout(60, method="thread")
@pytest.mark.parametrize("n,length", [(1, 1), (16, 32), (93, 192), (97, 200), (256, 512), (257, 540), (270, 540),
                                      (547, 1125), (1094, 2250), (2047, 4096), (2048, 4096), (2049, 4096), (1 << 30, 4096)])
def test_default_padded_length(n, length):
    """Up to 256 cells the lengths chosen before; above, the smallest 5-smooth length of at least 2n - 1 whose
    L / (largest radix) is at most 512 (1094 cells: 2187 = 3^7 has 729, 2250 = 6 5 5 5 3 has 375)."""
    import ctypes

    from paper_0704_0037_amd import dda
    assert getattr(dda.lib(), "_ZN3dda11default_padEi")(ctypes.c_int(n)) == length


def test_qmr_closes_late_only_where_a_product_is_short(tmp_path):
    """The extra product of a right-hand side that stops is short for one vector and for few vectors on
    specialized lengths; elsewhere it costs more than the launches it saves (measured beside the rule)."""
    out = _run(tmp_path, """
#include <cstdio>
#include "ctx.hpp"
int main() {
    const int c[][4] = {{1, 1, 24, 32}, {32, 1, 60, 64}, {7, 8, 32, 32}, {31, 2, 60, 60}, {22, 4, 48, 48},
                        {33, 1, 64, 64}, {22, 8, 48, 48}, {31, 8, 60, 60}, {1, 64, 15, 15}, {3, 2, 24, 32}, {3, 2, 32, 24}};
    for (auto &q : c) std::printf("%d ", (int)dda::qmr_closes_late(q[0], q[1], q[2], q[2], q[3]));
}
""")
    assert out == ["1"] * 5 + ["0"] * 6
