"""What tests of results cannot see, read from the sources.

The kernels' memory: an object is read with the scalar type that it was written with.  (Strict aliasing is on: a list of 16-bit
entries that is read through a pointer to 32-bit ones may be read before it is written.  Vector types may alias anything.)

The parity hook of the 4-bit products: it runs the product that the Selection-Pass runs, so there is one."""
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


def test_the_products_hook_and_the_selection_share_their_product():
    with open(os.path.join(CSRC, "select.hip")) as f:
        text = f.read()
    assert len(re.findall(r"__builtin_amdgcn_mfma_scale_f32_\w+\(", text)) == 1
    assert len(re.findall(r"\bqk_fp6\(", text)) == 3      # its definition, the Selection-Pass and the hook
