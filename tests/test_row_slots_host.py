"""Host-only check of the slot rule for sums over the wavefronts that share a row (csrc/common.hip.h): one barrier per sum is
enough exactly when no two consecutive sums of a workgroup's walk use the same slot, whatever the number of sums per row -
LayerNorm takes two per row, RMSNorm one.  The rule is compiled with the host compiler and walked; the kernel is read for
its use of it."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_14279_amd", "csrc")


@pytest.mark.parametrize("sums_per_row", [1, 2])
def test_consecutive_sums_use_different_slots(tmp_path, sums_per_row):
    text = open(os.path.join(CSRC, "common.hip.h")).read()
    rule = re.search(r"constexpr int row_sum_slot\(.*?\}\n", text, re.S).group(0)
    src, exe = tmp_path / "slots.cpp", tmp_path / "slots"
    src.write_text("#include <cstdio>\n" + rule + "int main() { for (int t = 0; t < 40; t++) for (int k = 0; k < %d; k++) "
                   "std::printf(\"%%d \", row_sum_slot(%d, t, k)); }\n" % (sums_per_row, sums_per_row))
    subprocess.run(["g++", "-std=c++17", str(src), "-o", str(exe)], check=True)
    slots = [int(v) for v in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()]
    assert len(slots) == 40 * sums_per_row and set(slots) == {0, 1}
    assert all(a != b for a, b in zip(slots, slots[1:]))


def test_the_normalisation_takes_its_slots_from_the_rule():
    text = open(os.path.join(CSRC, "rowwise.hip")).read()
    body = text[text.index("void f2_rows_kernel("):text.index("wg_sum2(C& a, C& b")]
    assert body.count("row_sum_slot(ACT == ACT_RMS ? 1 : 2, trip, k)") == 1 and body.count("trip++") == 1
    assert set(re.findall(r"pair\[(\w+)\]\[", body)) == {"2", "slot"}     # its declaration, and the rule's slot everywhere else
