"""What the library reads from the environment: tuning overrides named REDUCE_*, in the code that
picks launch shapes and reports tuning.  No kernel launch of the batched path depends on one."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2008_11486_amd", "csrc")


def test_only_named_overrides_are_read():
    read = {}
    for f in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, f)) as src:
            for name in re.findall(r'(?:getenv|env_int)\(\s*"([^"]*)"', src.read()):
                read.setdefault(f, set()).add(name)
    assert all(n.startswith("REDUCE_") for names in read.values() for n in names), read
    assert set(read) == {"combine.hip", "plan.cpp", "tune.cpp"}, read
