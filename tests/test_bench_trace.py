"""bench.py's summary of a kernel trace (host only): it finds the run's steps by the kernel that
opens one, and says so where it cannot."""
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)
import bench  # noqa: E402

OPENS = "void wam::(anonymous namespace)::gemv_kernel<1, 2, true>(int, int, int, float const*)"
LAYER = "void wam::(anonymous namespace)::gemv_kernel<1, 4, false>(int, int, int, float const*)"
GEMM = "void wam::(anonymous namespace)::gemm_nt<wam::(anonymous namespace)::Cfg<64, 64, 64, 4, 2, 2, 2, 2, 1, 1>, 0>(wam::GemmArgs, int, int)"


def write_trace(path, names):
    with open(path / "t_kernel_trace.csv", "w") as f:
        f.write('"Kernel_Name","Start_Timestamp","End_Timestamp","Grid_Size_X"\n')
        for i, n in enumerate(names):
            f.write(f'"{n}",{i * 10000000},{i * 10000000 + 2000000},64\n')


def test_per_step_times_leave_the_set_up_out(tmp_path, capsys):
    write_trace(tmp_path, [GEMM] * 5 + [OPENS, LAYER, GEMM] * 4)
    bench.trace_summary(str(tmp_path), 2)
    out = capsys.readouterr().out
    assert "over the last 2 steps: 6.00 ms" in out
    row = next(line for line in out.splitlines() if "gemm_nt" in line)
    assert row.rstrip().endswith("| 2.000 |")


def test_too_few_steps_are_an_error(tmp_path):
    write_trace(tmp_path, [GEMM] * 5 + [OPENS, LAYER, GEMM])
    with pytest.raises(SystemExit, match="1 steps in the trace"):
        bench.trace_summary(str(tmp_path), 2)


def test_the_library_has_the_kernel_that_opens_a_step():
    """The kernels' names as the library registers them, one template argument list per batch."""
    with open(os.path.join(ROOT, "paper_2602_15922_amd", "libwamdit.so"), "rb") as f:
        names = set(re.findall(rb"gemv_kernelILi(\d+)ELi(\d+)ELb1EE", f.read()))
    assert len(names) == 8
    for b, rows in names:
        assert bench.STEP_OPENS.search(f"void gemv_kernel<{int(b)}, {int(rows)}, true>")
