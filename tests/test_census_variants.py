"""The neighbour census is built with the page, lists and registers of every
pass that it stands for: for each FORCE and GRADIENT variant of the pair
kernel in the library there is the same variant as a census."""
import re
import shutil
import subprocess

import pytest

from paper_2310_03596_amd import _lib


def test_every_pass_has_its_census():
    if shutil.which("nm") is None:
        pytest.skip("no nm")
    names = subprocess.run(["nm", "-C", _lib.LIB_PATH], capture_output=True, text=True, check=True).stdout
    # k_pairs<real, pass, solid, targets per wavefront, census>; passes 0 (FORCE) and 1 (GRADIENT)
    found = set(re.findall(r"k_pairs<(\w+), (\d), (\w+), (\d+), (\w+)>", names))
    passes = {v[:4] for v in found if v[4] == "false" and v[1] in "01"}
    assert len(passes) == 2 * 3 * 3, sorted(found)   # forms; fluid FORCE, solid FORCE, GRADIENT; widths
    assert {v[:4] for v in found if v[4] == "true"} == passes
