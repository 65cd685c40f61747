"""The autotuner tries only launch fields that a kernel launch reads, and only
values that the library accepts (a field without effect can win by noise alone)."""

import glob
import os
import re

from paper_2409_15615_amd import kmg, tune

CSRC = os.path.join(os.path.dirname(os.path.abspath(kmg.__file__)), "csrc")


def test_every_field_is_read():
    text = "".join(open(p).read() for p in glob.glob(os.path.join(CSRC, "*.hip")) if not p.endswith("tuning.hip"))
    read = set(re.findall(r"tuning\(\)\.(\w+)", text))
    for alias in re.findall(r"const Tuning& (\w+) = tuning\(\);", text):
        read |= set(re.findall(rf"\b{alias}\.(\w+)", text)) & set(kmg.TUNING_FIELDS)
    assert set(tune.SPACE) <= read, set(tune.SPACE) - read
    assert set(tune.SPACE) == read & set(kmg.TUNING_FIELDS)


def test_every_value_is_accepted():
    try:
        for field, values in tune.SPACE.items():
            default = kmg.get_tuning()[field]
            assert default in values
            for v in values:
                kmg.set_tuning({field: v})
                assert kmg.get_tuning()[field] == v
            kmg.set_tuning(None)
    finally:
        kmg.set_tuning(None)
