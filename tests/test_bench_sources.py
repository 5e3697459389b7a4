"""The counter summaries that the bench reports are tied to the sources of the
kernels that it names: the file that defines a kernel, that of its caller and all
they include (the public header apart)."""
import glob
import os
import re

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1202_2462_amd", "csrc")


def with_includes(names):
    seen, todo = set(), list(names)
    while todo:
        n = todo.pop()
        if n not in seen:
            seen.add(n)
            with open(os.path.join(CSRC, n)) as f:
                todo += re.findall(r'#include "([^"/]+)"', f.read())
    return seen


def defining_file(kernel):
    found = [f for f in glob.glob(os.path.join(CSRC, "*.hip")) if re.search(r"\b%s\(\s" % kernel, open(f).read())]
    assert len(found) == 1, (kernel, found)
    return os.path.basename(found[0])


def test_sources_of_the_named_kernels():
    for kernel, callers, listed in ((bench.SAP_KERNEL, ["sap.hip"], bench.SAP_SOURCES),
                                    (bench.COARSE_KERNEL, [], bench.COARSE_SOURCES)):
        need = with_includes([defining_file(kernel)] + callers)
        assert need <= {os.path.basename(f) for f in listed}, (kernel, need)


def test_summaries_are_of_the_named_kernels():
    for kernel, path in ((bench.SAP_KERNEL, bench.TRAFFIC_FILE), (bench.COARSE_KERNEL, bench.COARSE_TRAFFIC_FILE)):
        if os.path.exists(path):
            with open(path) as f:
                assert kernel in f.readline()
