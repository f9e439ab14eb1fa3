"""The sort's kernels take a count that no kernel running beside them can change."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2301_07331_amd", "csrc")

CHECK = """
#include <type_traits>
#include "hlc_kernels.hpp"
// (a member that points at a flag: read by some waves before it is set and by others after)
template <class T, class = void> struct has_flag : std::false_type {};
template <class T> struct has_flag<T, std::void_t<decltype(std::declval<T&>().none)>> : std::true_type {};
template <class T, class = void> struct has_over : std::false_type {};
template <class T> struct has_over<T, std::void_t<decltype(std::declval<T&>().over)>> : std::true_type {};
static_assert(!has_flag<decltype(hlc::BucketIn::cnt)>::value, "the sort's own count");
static_assert(!has_over<hlc::BucketIn>::value, "the sort's own input");
"""


def test_sort_count_has_no_flag(tmp_path):
    from paper_2301_07331_amd import build_lib
    src = tmp_path / "check.hip"
    src.write_text(CHECK)
    run = subprocess.run([build_lib.HIPCC, *build_lib.FLAGS, "-I", CSRC, "-fsyntax-only", str(src)],
                         capture_output=True, text=True)
    assert run.returncode == 0, run.stderr
