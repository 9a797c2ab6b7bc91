"""Properties of the kernel sources that no run can show: a wave's LDS
accesses happen to execute in order, so a missing fence changes nothing until
the compiler moves an access."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2512_08478_amd", "csrc")


def test_shared_sh_rows_are_fenced():
    """Lanes that stage SH rows in LDS store vectors of other lanes' rows: a
    barrier or a fence of the wave stands between those stores and the reads of a
    row, and in the kernel that stages half a wave's rows at a time also between
    the reads of one half and the stores of the next."""
    txt = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, "preprocess.hip")).read())
    token = (r"(?P<fence>wave_lds_sync\(\)|__syncthreads\(\))|(?P<store>\b(?:buf|rows|s_sh)\[[^;=]*\] = )|"
             r"(?P<read>row_colour<DEG>\((?:buf|rows)|LdsRow<DEG>\{s_sh)")

    def events(text):
        return [m.lastgroup for m in re.finditer(token, text)]
    every = events(txt)
    assert every.count("store") == 4 and every.count("read") == 3
    assert ("store", "read") not in list(zip(every, every[1:]))
    halves = txt[txt.index("preprocess_block("):]
    assert events(halves[:halves.index("block_counts(")]) == ["store", "fence", "read", "fence"]
