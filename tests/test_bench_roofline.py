"""The benchmark's roofline line states the rule of the kernel that it names: the
stated sum of the stated sizes is the bytes that the duration is divided by, and the
per-mode records are the solve's alone."""
import re

import pytest


@pytest.mark.parametrize("workload", ["couette_48x65x48_re1000_dt100",
                                      "couette_96x97x96_re2000_dt100"])
@pytest.mark.parametrize("fused", [False, True])
def test_rule_gives_the_bytes(workload, fused):
    import bench
    w = bench.WORKLOADS[workload]
    ab = bench.algorithmic_bytes(w, fused=fused)
    rules = set()
    for kernel, alg in ab.items():
        b, rule, record = bench.roofline_bytes(kernel, w, fused)
        assert b == alg
        terms = rule.split(" (")[0]
        sizes = {n: int(v) for n, v in re.findall(r"(\w) = (\d+) B", rule)}
        assert sum(int(c) * sizes[n] for c, n in re.findall(r"(\d+) (\w)", terms)) == alg, rule
        assert record == (bench.record_bytes(w) if kernel == "k_stokes_solve" else None)
        rules.add(rule)
    assert len(rules) == len(ab)
