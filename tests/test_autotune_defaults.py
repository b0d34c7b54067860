"""The tuner times a batch's defaults by setting them, and leaves out of the table what equals
them: they have to be the library's own."""
import os
import re

from paper_2004_08227_amd import autotune as A

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2004_08227_amd", "csrc", "batch.cpp")


def test_batch_defaults_are_the_librarys():
    text = open(SRC).read()

    def value(name):
        return [float(x) for x in re.search(rf"\b{name}\s*(?:\[\d\])?\s*=\s*\{{?([^;}}]*)\}}?;", text).group(1).split(",")]

    lib = dict(zip(("wave_edge16_us", "wave_edge32_us", "wave_edge64_us"), value("wv_edge_us")))
    lib["wave_lat_mb_us"], = value("wv_lat_mb_us")
    lib["wave_lat_lds_us"], = value("wv_lat_lds_us")
    for key, v in lib.items():
        assert A.BATCH_DEFAULTS[key] == v, key
    for key, choices in A.BATCH_CHOICES.items():
        assert A.BATCH_DEFAULTS[key] in choices, key
