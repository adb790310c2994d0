"""What the compiler may assume about the kernels' memory: an object is read with the scalar type that it was written with.
(Strict aliasing is on: a list of 16-bit entries that is read through a pointer to 32-bit ones may be read before it is
written.  Vector types may alias anything.)"""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_24179_amd", "csrc")
PUN = re.compile(r"\*\s*\(\s*(const\s+)?(u?int\d+_t|unsigned|int|short|float|double)\s*(const\s*)?\*\s*\)\s*\(")


def test_no_scalar_is_read_through_another_scalar_type():
    found = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip"))):
        with open(path) as f:
            found += [f"{os.path.basename(path)}:{n}: {line.strip()}" for n, line in enumerate(f, 1) if PUN.search(line)]
    assert not found, found
