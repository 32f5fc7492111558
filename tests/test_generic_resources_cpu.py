"""Register, scratch and LDS budgets of the fp32-weight attention kernels (no
GPU), as test_resources_cpu.py has them for the others: no dynamic stack, no
spilled SGPRs, no occupancy target missed; no scratch but a few values in fp16
at 65 to 96 columns, whose four-block layout is held to 128 registers so that
two workgroups share a CU; every layout's workgroups fit a CU at all."""
import re

import pytest

from test_resources_cpu import _num, _parse, _report


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    return _report("fa_generic.hip", str(tmp_path_factory.mktemp("resources")))


def test_budgets(report):
    assert "failed to meet occupancy target" not in report
    kernels = _parse(report)
    layouts = set()
    for name, k in kernels.items():
        m = re.search(r"generic_kernelI(f|NS_\d+\w+?E).*?Li(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", name)
        assert m, name
        tin, DP, NSLOT, KSP, NB = m.group(1), *(int(m.group(i)) for i in range(2, 6))
        layouts.add((tin == "f", DP, NSLOT, KSP))
        assert k["Dynamic Stack"] == "False", name
        assert _num(k, "SGPRs Spill") == 0, name
        four_96 = tin != "f" and DP == 96 and NSLOT == 4
        scratch = _num(k, "ScratchSize [bytes/lane]")
        assert scratch <= (16 if four_96 and "f16_t" in tin else 0), (name, scratch)
        waves, occ = NSLOT * KSP, _num(k, "Occupancy [waves/SIMD]")
        assert 4 * occ >= waves * (2 if four_96 else 1), (name, occ)
        assert _num(k, "LDS Size [bytes/block]") * (2 if four_96 else 1) <= 160 * 1024, name
    assert {lay[1] for lay in layouts} == set(range(32, 257, 32))
    assert {lay[2:] for lay in layouts} == {(1, 4), (2, 4), (2, 2), (4, 2), (8, 1)}
