"""The bound that the sampling kernel puts on a token's Gumbel noise, for every
one of the 2^23 values the noise takes: never below it, by at least half of the
margin (2^-10) that its constant holds for rounding.  The two constants are
read from the kernel's source."""
import os
import re

import numpy as np

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2403_06988_amd", "csrc",
                      "dv_sample.hip")


def _fma(a, b, c):
    """Products of binary32 are exact in binary64; the sum rounds twice, which
    moves a result by one unit in the last place at most."""
    return (a.astype(np.float64) * np.float64(b) + np.asarray(c, np.float64)).astype(np.float32)


def _ln(x):
    bits = x.view(np.uint32)
    e = (bits >> 23).astype(np.int32) - 127
    mb = (bits & 0x007FFFFF) | 0x3F800000
    high = mb > 0x3FB504F3
    mb = np.where(high, mb - 0x00800000, mb).astype(np.uint32)
    e = e + high
    return (np.log(mb.view(np.float32).astype(np.float64)) + e * np.log(2.0)).astype(np.float32)


def test_gumbel_bound_holds_for_every_word():
    with open(SOURCE) as f:
        body = f.read().split("float gumbel_bound_of_word(uint32_t w)")[1].split("}")[0]
    slope, offset = (np.float32(float.fromhex(c)) for c in re.findall(r"(-?0x[0-9a-f.]+p[+-]\d+)f", body))
    worst = np.inf
    for start in range(0, 2**23, 2**20):
        k = np.arange(start, start + 2**20, dtype=np.uint32)
        u = ((2 * k + 1).astype(np.float64) * 2.0**-24).astype(np.float32)
        noise = -_ln(-_ln(u))
        for low in (0, 511):                       # the word's low bits do not enter the noise
            w = k << np.uint32(9) | np.uint32(low)
            f = (~(w | np.uint32(0xFF))).astype(np.float32)
            bound = _fma(f.view(np.uint32).astype(np.float32), slope, offset)
            worst = min(worst, float((bound.astype(np.float64) - noise).min()))
    assert worst >= 2.0**-11
