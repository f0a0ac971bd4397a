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


def spills():
    """Spilled vector registers of every kernel in the built library, from the metadata that the compiler leaves with it."""
    from paper_2603_02883_amd import build
    data, found = open(build.LIB, "rb").read(), {}
    # per kernel a map with its keys in order: .symbol "<name>.kd", ..., .vgpr_spill_count <integer>
    for m in re.finditer(rb"\.symbol(?:[\xa0-\xbf]|\xd9.|\xda..)(\w+)\.kd.{0,80}?\.vgpr_spill_count([\x00-\x7f]|\xcc.|\xcd..)", data, re.S):
        count = m.group(2)
        found[m.group(1).decode()] = int.from_bytes(count[1:], "big") if len(count) > 1 else count[0]
    return found


def test_kernels_keep_their_values_in_registers():
    """A spilled value's reload waits for every load in flight.  Those that still spill are GeLU in block 16 with 16 groups, on 16
    wavefronts, one LayerNorm of six chunks per lane with lists, and one register of one with one chunk and both restrictions."""
    found = spills()
    assert len(found) > 300 and any("layernorm" in k for k in found) and any("attention" in k for k in found)
    allowed = {"gelu_quantize_kernelILi16ELi16ELb0ELb1E": 8, "gelu_quantize_kernelILi16ELi16ELb1ELb0E": 8, "gelu_quantize_kernelILi16ELi16ELb1ELb1E": 4,
               "layernorm_quantize_kernelILi6ELi16ELi16ELb0ELb1E": 4, "layernorm_quantize_kernelILi1ELi16ELi16ELb1ELb1E": 1}
    over = {k: n for k, n in found.items() if n > max([v for a, v in allowed.items() if a in k], default=0)}
    assert not over


def test_kernel_arguments_fit_a_launch():
    """The runtime carries 112 bytes of kernel arguments with a launch and allocates for more; what a kernel reads of its own launch
    (its grid's size, say) comes as 256 more."""
    from paper_2603_02883_amd import build
    data, sizes = open(build.LIB, "rb").read(), []
    for m in re.finditer(rb"\.kernarg_segment_size([\x00-\x7f]|\xcc.|\xcd..)", data, re.S):
        count = m.group(1)
        sizes.append(int.from_bytes(count[1:], "big") if len(count) > 1 else count[0])
    assert len(sizes) == len(spills()) > 300 and max(sizes) <= 112
