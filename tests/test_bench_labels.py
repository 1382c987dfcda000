"""CPU check: the benchmark has a label for every kernel family the library can report."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_kernel_family_has_a_label():
    import bench
    with open(os.path.join(ROOT, "paper_2506_17870_amd", "csrc", "nq_gemm.hip")) as f:
        families = {int(n) for n in re.findall(r"g_last_family = (\d+);", f.read())} - {0}
    assert families == set(bench.FAMILY)


def test_a_launch_reports_the_kernel_it_launches():
    import bench
    with open(os.path.join(ROOT, "paper_2506_17870_amd", "csrc", "nq_gemm.hip")) as f:
        text = f.read()
    seen = set()
    for before, launcher in re.findall(r"(.*?)NQ_DISPATCH_HL\(h, l, launch_nested_(\w+),", text, re.S):
        kernel = "k_nested_" + launcher.replace("_batch", "")
        numbers = {int(n) for n in re.findall(r"g_last_family = (\d+);", before)} - {0}
        assert numbers, launcher
        for n in numbers:
            assert any(kernel.endswith(part) for part in bench.FAMILY[n].split(" / ")), (launcher, n)
        seen |= numbers
    assert seen == set(bench.FAMILY)
