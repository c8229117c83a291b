"""Device records that the host only addresses: a member that a kernel loads
as a 16-byte (re, im) pair lies on a 16-byte boundary of the record, whose
buffer is at least so aligned. Checked by the compiler, without a GPU."""
import subprocess

from paper_1204_5463_amd import build as B

SOURCE = """
#include <type_traits>
#include "dw_kernels.hpp"
#include "dw_types.hpp"
using namespace dw;
static_assert(std::is_same<decltype(&blas_rms_scale), dw_status (*)(const void*, int, long long, bool, double*,
                                                                    RmsScale*, hipStream_t)>::value, "");
static_assert(alignof(RmsScale) >= alignof(s64) && offsetof(RmsScale, inverse) % alignof(s64) == 0, "");
"""


def test_rms_scale_inverse_is_a_pair(tmp_path):
    src = tmp_path / "layout.hip"
    src.write_text(SOURCE)
    p = subprocess.run([B.HIPCC] + B.COMMON + ["-fsyntax-only", "--cuda-host-only", str(src)], capture_output=True,
                       text=True)
    assert p.returncode == 0, p.stderr
