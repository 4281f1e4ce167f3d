"""A right-hand side's bookkeeping folds the 64 counter lines with one lane
each: every kernel that runs it does so with a whole wave.  (On the device a
launch with fewer lanes reads lanes that do not run, which is undefined but
mostly zero, so that nothing shows.)"""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_22269_amd", "csrc")


def test_bookkeeping_runs_in_a_whole_wave():
    src = open(os.path.join(CSRC, "grid.hip")).read()
    launches = re.findall(r"hipLaunchKernelGGL\(k_prep,\s*dim3\((\w+)\),\s*dim3\((\w+)\)", src)
    assert launches and all(d == ("1", "64") for d in launches), launches
    for other in ("k_hash_f64<2>", "k_hash_f64<3>", "k_hash_packed"):
        for grid, block in re.findall(r"hipLaunchKernelGGL\(" + re.escape(other) +
                                      r",\s*dim3\(([^,]*)\),\s*dim3\(([^,]*)\)", src):
            assert block == "kBlock", (other, grid, block)
    # its first wave, not single threads of it
    assert re.findall(r"if \(prep\.on && i < (\d+)\) run_prep", src) == ["64", "64"]
