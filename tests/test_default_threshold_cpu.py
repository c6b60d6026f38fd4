"""The default det thresholds stand in the library, in its header's documentation
and in the benchmark's report: the three must say the same."""
import os
import re

from paper_2411_19901_amd import build

# (log2 of the entries below which it holds, threshold); the last holds for the rest
def library():
    with open(os.path.join(build.CSRC, "capi.hip")) as f:
        body = re.search(r"kDetSteps\[\] = \{(.*?)\};", f.read(), re.S).group(1)
    steps = re.findall(r"\{\(int64_t\)1 << (\d+), (\d+)\}", body)
    last = re.search(r"\{INT64_MAX, (\d+)\}", body).group(1)
    return [(int(e), int(s)) for e, s in steps], int(last)


def test_header():
    with open(os.path.join(build.INCLUDE, "lpa.h")) as f:
        text = " ".join(re.sub(r"^ *\*? ?", "", x) for x in f)
    text = re.search(r"det (\d+ below .*?else \d+)\)", " ".join(text.split())).group(1)
    steps = [(int(e), int(s)) for s, e in re.findall(r"(\d+) below 2\^(\d+)", text)]
    assert (steps, int(re.search(r"else (\d+)", text).group(1))) == library()


def test_benchmark():
    with open(os.path.join(build.ROOT, "bench.py")) as f:
        text, last = re.search(r"det_default = next\((.*?), (\d+)\)\n", f.read(), re.S).groups()
    steps = [(int(e), int(s)) for e, s in re.findall(r"\((\d+), (\d+)\)", text)]
    assert (steps, int(last)) == library()
