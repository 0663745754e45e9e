"""CPU: the bench's counter summary names the kernels as they are in the
sources and adds up a kernel's instantiations."""
import glob
import inspect
import os
import re
import sys

HERE = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, HERE)
import bench  # noqa: E402

from .test_bench_tools import _db  # noqa: E402

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


def test_counter_summary_adds_instantiations(tmp_path):
    rows = [("lk::k_batch_apply_old(lk::BatchArgs)", 0, 10, 0),
            ("void lk::k_move_async<4, 512, false>(lk::MoveArgs)", 20, 30, 1),
            ("void lk::k_move_async<4, 512, true>(lk::MoveArgs)", 40, 50, 2),
            ("void lk::k_move_async<4, 512, true>(lk::MoveArgs)", 60, 70, 3),
            ("void lk::k_mod_intra<double>(long const*, ...)", 80, 90, 4)]
    db = str(tmp_path / "c.db")
    _db(db, rows, [(1, "TCC_ATOMIC_sum", 100.0), (2, "TCC_ATOMIC_sum", 30.0), (3, "TCC_ATOMIC_sum", 7.0)])
    md = bench.summarize_counters(db, "cmd")
    assert "| TCC_ATOMIC_sum | 137 |" in md and md.count("k_move_async") == 1
