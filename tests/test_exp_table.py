"""The table and the polynomial of the sampled acceptance's short exponential (csrc/tree.hip), on the CPU."""
import os
import re
import struct
from decimal import Decimal, getcontext

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = open(os.path.join(ROOT, "paper_2409_00142_amd", "csrc", "tree.hip")).read()


def test_table_of_powers():
    """Entry j is 2^(j/128) rounded to the nearest double, less j units of 2^-7 in the exponent field (its high word less j << 13), which
    adding n << 13 for n = 128 e + j turns into the exponent e."""
    getcontext().prec = 60
    body = re.search(r"kVsExp\[kVsExpSize\] = \{(.*?)\};", SOURCE, re.S).group(1)
    table = [int(x, 16) for x in re.findall(r"0x([0-9a-f]{16})ull", body)]
    assert len(table) == 128
    for j, bits in enumerate(table):
        exact = (Decimal(2).ln() * j / 128).exp()
        nearest = struct.unpack("<Q", struct.pack("<d", float(exact)))[0]
        assert bits == nearest - (j << (13 + 32)), j


def test_polynomial():
    """1 + f p(f) against 2^f over |f| <= 1/256: 2e-16, in exact arithmetic on the coefficients as written."""
    getcontext().prec = 40
    body = SOURCE[SOURCE.index("double add_weight("):]
    first = re.search(r"double p = ([0-9.]+);", body)
    rest = re.findall(r"p = fma\(p, f, ([0-9.]+)\);", body[first.end():])[:4]
    assert rest[-1] == "1.0"
    c = [Decimal(float(x)) for x in [first.group(1)] + rest]
    worst = Decimal(0)
    for i in range(-256, 257):
        f = Decimal(i) / (256 * 256)
        p = Decimal(0)
        for x in c:
            p = p * f + x
        worst = max(worst, abs(p / (Decimal(2).ln() * f).exp() - 1))
    assert worst < Decimal("2e-16"), worst
