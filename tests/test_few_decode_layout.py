"""The few-blocks decoder extracts every array of a record in LDS at all B
positions, also in a partial block.  Its buffer has to hold the highest word
such a read touches: computed here from the oracle's streams whose partial
block has a record just under the longest that is decoded from LDS."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_10305_amd", "csrc")


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    """(longest record, {B: words of the buffer})"""
    d = tmp_path_factory.mktemp("layout")
    src, exe = d / "layout.cpp", d / "layout"
    src.write_text('#include <cstdio>\n#include "decode_layout.h"\n'
                   'int main() { std::printf("%u\\n", gpz::kFewRecWords);\n'
                   'for (unsigned B = 256; B <= 2048; B *= 2)\n'
                   '    std::printf("%u %u\\n", B, gpz::few_rec_room(B)); }\n')
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    return int(lines[0]), dict(tuple(map(int, x.split())) for x in lines[1:] if x)


def last_record(words, n, F, B):
    """The words of the last block's record."""
    nb = -(-n // B)
    lens = words[8 + 2 * (-(-nb // 64)) + F:][:nb]
    return words[words.size - int(lens[-1]):]


def highest_read(rec, nb, F, B):
    """Highest word of `rec` an extraction of all B positions reads."""
    def count(values, width):
        return (values * width + 31) // 32

    U, h1 = int(rec[0]) >> 2, int(rec[1])
    pos, top = 2 + count(U, h1 & 31) + count(U, (h1 >> 5) & 31), 0
    for _ in range(F):
        w, nout = int(rec[pos + 1]) & 31, int(rec[pos + 1]) >> 5
        top = max(top, pos + 2 + ((B - 1) * w // 32) + 1)
        pos += 2 + count(nb, w) + 2 * nout
    assert pos == rec.size
    return top


@pytest.mark.parametrize("B,part,F,eb", [(2048, 1433, 6, 1e-4), (2048, 614, 8, 1e-6),
                                         (1024, 512, 10, 1e-6), (256, 250, 20, 1e-6),
                                         (512, 500, 10, 1e-6)])
def test_reads_of_a_partial_block_stay_in_the_buffer(orc, layout, B, part, F, eb):
    longest, room = layout
    rng = np.random.default_rng(B + part)
    n = B + part
    host = [rng.standard_normal(n).astype(np.float32) for _ in range(F)]
    words = orc.compress(host, eb, B=B)[0].view(np.uint32)
    rec = last_record(words, n, F, B)
    assert int(rec[0]) & 3 == 0 and 0.75 * longest < rec.size <= longest, rec.size
    assert highest_read(rec, part, F, B) < room[B]


@pytest.mark.parametrize("B", [256, 512, 1024, 2048])
def test_any_record_fits(layout, B):
    """The last array may begin at the longest record's end (an array of one
    value, 24 bits wide); staging fills whole steps up to the longest record."""
    longest, room = layout
    assert longest + ((B - 1) * 24) // 32 + 1 < room[B]
