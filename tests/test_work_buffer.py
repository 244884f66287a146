"""The work buffer's form of a float64 tangent pass (csrc/work_buffer.h): host
logic, compiled and run on the CPU."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_10357_amd", "csrc")


def run_cpp(tmp_path, body):
    src = tmp_path / "t.cpp"
    src.write_text('#include <cstdio>\n#include "work_buffer.h"\nusing namespace tlfea;\nint main() {\n' + body + "\n}\n")
    exe = tmp_path / "t"
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()


# (rows, records, capacity) -> rows taken
@pytest.mark.parametrize("rows,records,cap,want", [
    (768, 384, 0, 1), (768, 384, 383, 1),            # nothing yet, or a force-sized buffer
    (768, 384, 384, 0), (768, 384, 767, 0),          # sized for the records: it stays
    (768, 384, 768, 1), (768, 384, 4096, 1),         # sized for the rows
    (520, 880, 0, 1), (520, 880, 519, 1), (520, 880, 520, 1), (520, 880, 880, 1),  # the rows are the smaller
])
def test_a_buffer_sized_for_records_stays(tmp_path, rows, records, cap, want):
    assert run_cpp(tmp_path, f'std::printf("%d\\n", (int)buffer_takes_rows({rows}, {records}, {cap}));') == [str(want)]


# (needed, smaller form, what the device has) -> status, bytes asked for in turn
@pytest.mark.parametrize("need,smaller,have,want", [
    (768, 384, 1000, "0 768"), (768, 384, 768, "0 768"),
    (768, 384, 767, "0 768 384"), (768, 384, 384, "0 768 384"),  # the records fit
    (768, 384, 383, "-5 768 384"),                               # nothing does: TLFEA_ERR_NOMEM
    (520, 880, 519, "-5 520"), (768, 768, 100, "-5 768"),        # no smaller form
])
def test_without_memory_for_the_rows_the_records_are_taken(tmp_path, need, smaller, have, want):
    body = f"""
  size_t asked[4]; int n = 0;
  const int rc = take_buffer({need}, {smaller}, [&](size_t b) {{
    asked[n++] = b;
    return b <= {have} ? TLFEA_OK : TLFEA_ERR_NOMEM;
  }});
  std::printf("%d", rc);
  for (int i = 0; i < n; ++i) std::printf(" %zu", asked[i]);
"""
    assert run_cpp(tmp_path, body) == want.split()


def test_other_errors_are_not_retried(tmp_path):
    body = """
  int n = 0;
  const int rc = take_buffer(768, 384, [&](size_t) { ++n; return TLFEA_ERR_HIP; });
  std::printf("%d %d", rc, n);
"""
    assert run_cpp(tmp_path, body) == ["-4", "1"]
