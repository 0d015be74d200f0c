"""The limits up to which a row-broadcast tile takes a whole block, as the source
has them, and that the tests of the two forms lie on either side of them."""
import os
import re

import test_gpu_split as split

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_both_forms_are_tested_at_their_limits():
    text = open(os.path.join(ROOT, "paper_1811_05474_amd", "csrc", "rwpt_kernels.h")).read()
    m = re.search(r"split_tiles_for\(double nb\) \{ return nb > ([\d.]+) \? (\d+) : (\d+); \}", text)
    dense, wide, narrow = float(m.group(1)), int(m.group(2)), int(m.group(3))
    cases = split.test_neighbour_sets_and_masses.pytestmark[-1].args[1]
    limit = [(c[1], wide if c[2] > dense else narrow) for c in cases]
    for most in (wide, narrow):
        tiles = {t for t, at in limit if at == most}
        assert {most, most + 1} <= tiles, (most, tiles)
    assert any(t < 16 for t, _ in limit)
