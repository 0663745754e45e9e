"""CPU: the bench's counter summary names the kernels as they are in the
sources."""
import glob
import inspect
import os
import re
import sys

HERE = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, HERE)
import bench  # noqa: E402

DEFAULT = inspect.signature(bench.summarize_counters).parameters["kernels"].default


def test_counter_summary_names_existing_kernels():
    """rocprofv3 lists a kernel template's instantiations with their return
    type, other kernels without; each listed form is one of the sources'."""
    src = "".join(open(p).read() for p in glob.glob(os.path.join(HERE, "paper_2405_11658_amd", "csrc", "*.hip")))
    forms = set()
    for m in re.finditer(r"(template <[^;{}]*>\s*)?__global__[^;{}]*?\bvoid (k_\w+)\(", src):
        forms.add(("void lk::" if m.group(1) else "lk::") + m.group(2))
    assert "lk::k_agg_group" in forms and "void lk::k_move_async" in forms
    for name in DEFAULT:
        assert name in forms, name
