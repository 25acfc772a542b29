"""Kernels whose partial results are counted at compile time: a count that has no kernel launches nothing and makes the call fail."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2408_00264_amd", "csrc")

MAIN = r"""
#include <cstdio>
int main() {
  for (int n = -1; n <= 10; ++n) {
    int got = -1;
    g_not_launched = nullptr;
    with_count<%d, %d>(n, [&](auto c) { got = decltype(c)::value; });
    printf("%%d,%%d ", got, g_not_launched != nullptr);
  }
}
"""


def test_counts_without_a_kernel(tmp_path):
    head = open(os.path.join(CSRC, "clover_internal.h")).read()
    text = "#include <type_traits>\n" + re.search(r"^inline thread_local const char\* g_not_launched.*?^}", head, re.S | re.M)[0]
    for lo, hi in ((0, 8), (1, 8), (3, 3)):
        (tmp_path / "k.cpp").write_text(text + MAIN % (lo, hi))
        subprocess.run(["g++", "-std=c++17", str(tmp_path / "k.cpp"), "-o", str(tmp_path / "k")], check=True)
        out = subprocess.run([str(tmp_path / "k")], capture_output=True, text=True, check=True).stdout.split()
        assert out == [f"{n},0" if lo <= n <= hi else "-1,1" for n in range(-1, 11)], (lo, hi, out)


def test_calls_report_what_was_not_launched():
    """every use of the count goes through an entry point that asks"""
    api = open(os.path.join(CSRC, "clover_api.hip")).read()
    body = re.search(r"^int finish\(.*?^}", api, re.S | re.M)[0]
    assert "g_not_launched" in body and "CLOVER_E_STATE" in body
    ops = api[api.index("size_t clover_op_gemm_scratch_bytes"):]          # (the operators have no context and end without finish)
    refusing = set()   # launchers that may launch nothing
    for f in sorted(os.listdir(CSRC)):
        if f.endswith((".hip", ".h")):
            for m in re.finditer(r"^(?:template <[^\n]*>\n)?(?:static )?(?:inline )?void (launch_\w+)\(.*?^}", open(os.path.join(CSRC, f)).read(), re.S | re.M):
                if re.search(r"with_count<|g_not_launched =", m[0]):
                    refusing.add(m[1])
    assert refusing >= {"launch_reduce_add_norm", "launch_rope_kv_planes", "launch_rope_kv_parts", "launch_tile_few"}, refusing   # (the search finds them)
    tile = open(os.path.join(CSRC, "gemm_tile.h")).read()                 # (of the GEMM's forms only the QKV projection's refuses)
    assert tile.count("g_not_launched") == 1 and re.search(r"if constexpr \(EPI != 3\) {[^}]*} else g_not_launched =", tile)
    for name in refusing - {"launch_tile_few"} | {"launch_gemm_qkv"}:
        assert name + "(" not in ops, name
