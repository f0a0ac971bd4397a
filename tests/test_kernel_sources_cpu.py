"""Properties of the kernels that are visible in their sources and in the built library, without a GPU."""

import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_02883_amd", "csrc")


def test_biased_offsets_are_summed_before_they_meet_a_pointer():
    """A table offset with the bins' bias taken off is a number modulo 2^32: by itself it lies 4 GiB behind the table, so the
    bin's part has to be added in 32 bits first."""
    sources = {os.path.basename(f): open(f).read() for f in glob.glob(os.path.join(CSRC, "*.h*"))}
    biased = set(re.findall(r"(\w+) = [^;]*- kBinBias \*", "".join(sources.values())))
    assert biased == {"row_base", "pbase"}
    for name, text in sources.items():
        for line in text.splitlines():
            code = line.split("//")[0]
            # pointer + offset, or offset + pointer, without a parenthesis or a function around the offset's own sum
            assert not re.search(r"\b(lds|reinterpret_cast<[^>]*>\([^)]*\))\s*\+\s*((K|M)\.)?(row_base|pbase)\b", code), (name, line)
            assert not re.search(r"\b(row_base|pbase)\s*\+\s*lds\b", code), (name, line)
