"""bench.py prices a kernel by what the plan took, not by its precision."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_executed_flop_follows_the_plans_kernels():
    sys.path.insert(0, ROOT)
    import bench
    import paper_2502_17789_amd as aidg

    def per(grid, degrid, split=0):
        e = bench.flop_executed({"grid_kernel": grid, "degrid_kernel": degrid, "w_terms": 1,
                                 "n_subgrids_split": split}, 100)
        return [(e[k]["flop"], e[k]["unit"]) for k in ("grid_dft", "degrid_dft")]
    assert per(aidg.KERNEL_GENERAL, aidg.KERNEL_GENERAL) == [(19, "vector")] * 2
    assert per(aidg.KERNEL_MATRIX, aidg.KERNEL_GENERAL) == [(128, "fp16 matrix cores"), (19, "vector")]
    assert per(aidg.KERNEL_MATRIX_WIDE, aidg.KERNEL_MATRIX, 25) == [(192, "fp16 matrix cores"), (144, "fp16 matrix cores")]
