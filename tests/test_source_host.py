"""Rules that the device sources keep, read from their text."""
import glob
import os
import re

from paper_2512_13368_amd import build


def test_values_are_not_reached_through_pointers_to_another_scalar_type():
    # the compiler may take a float and an integer at one address for unrelated, unless its file says otherwise (-fno-strict-aliasing): a
    # wait that names a float's register as an integer would then wait for nothing.  (Vectors such as uint4 may alias anything.)
    found = []
    for path in sorted(glob.glob(os.path.join(build.CSRC, "*.hip"))):
        if "-fno-strict-aliasing" in build.SOURCES[os.path.basename(path)]:
            continue
        for n, line in enumerate(open(path), 1):
            if re.search(r"reinterpret_cast<(unsigned|int|float|unsigned long long) \*>\((this\b|&\w+\)|bits|ws\.)", line):
                found.append(f"{os.path.basename(path)}:{n}: {line.strip()}")
    assert not found, found
