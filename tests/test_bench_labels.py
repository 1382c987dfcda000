"""CPU check: the benchmark has a label for every kernel family the library can report."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_kernel_family_has_a_label():
    import bench
    with open(os.path.join(ROOT, "paper_2506_17870_amd", "csrc", "nq_gemm.hip")) as f:
        families = {int(n) for n in re.findall(r"g_last_family = (\d+);", f.read())} - {0}
    assert families == set(bench.FAMILY)
