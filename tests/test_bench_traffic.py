"""The sources that bench.py's committed HBM counters are tied to."""
import os

import bench

CSRC = os.path.join(os.path.dirname(os.path.abspath(bench.__file__)), "paper_1402_6081_amd", "csrc")


def _defines(name):
    """The sources that define `name` (a line that begins with its declaration or body)."""
    out = []
    for f in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, f)) as fh:
            if any(name + "(" in line and line.rstrip().endswith(("{", "}")) and not line.startswith(" ")
                   for line in fh):
                out.append(f)
    return out


def test_counters_lapse_with_the_rules_they_depend_on():
    """A step's counters are stale once a source that decides what its kernel moves has changed: the
    order and runs of the level-0 groups, the order of the M2L's parents and its variant, and the
    stride of the level-0 field spectra, which the inverse transform reads."""
    for rule, families in (("run_length", ["prod"]), ("order_groups", ["prod"]), ("order_parents", ["prod"]),
                           ("m2l_default", ["prod"]), ("field_items", ["prod", "fft"])):
        where = _defines(rule)
        assert len(where) == 1, (rule, where)
        for fam in families:
            assert where[0] in bench._SRC[fam], (rule, fam)
