"""bench.py names the kernel and the passes a workload runs (host logic)."""
import bench
import paper_1208_2407_amd as tsq


def test_small_meshes_left_to_the_library_report_the_tile_kernels():
    plan = tsq.Plan(256, 256, 0.1, "c128")
    passes, copy_back = plan.passes(100)
    assert bench.passes_report(plan, 100, True) == {
        "kernel": "tile_kernel", "steps_per_pass": round(100 / passes, 2), "passes_per_solve": passes,
        "copy_back": copy_back}
    assert plan.passes(100) == (passes, copy_back)  # the plan's choice is left as it was


def test_schedules_report_the_march():
    plan = tsq.Plan(256, 256, 0.1, "c128")
    plan.set_schedule(5, 0, 1, 1)
    march = {"kernel": "march_kernel", "steps_per_pass": 5, "segment_rows": 0, "pairs_per_lane": 1,
             "phase_store": "registers", "passes_per_solve": 20, "copy_back": False}
    assert bench.passes_report(plan, 100, False) == march
    big = tsq.Plan(4096, 4096, 0.1, "c128")
    assert bench.passes_report(big, 100, True) == march
