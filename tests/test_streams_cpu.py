"""The library's device work is enqueued on the caller's stream: no source clears
memory or launches a kernel on the null stream, which has no order with
a non-blocking stream.  (A host-only check of the sources: the races this prevents
show now and then only.)"""
import glob
import os
import re

import paper_2104_01196_amd as g

CSRC = os.path.join(os.path.dirname(g.__file__), "csrc")


def test_nothing_cleared_on_the_null_stream():
    """(hipMemcpy from host memory is complete when it returns; hipMemset of device memory need not be.)"""
    files = sorted(glob.glob(os.path.join(CSRC, "*.h*p")))
    assert len(files) >= 8
    for f in files:
        for k, line in enumerate(open(f).read().splitlines(), 1):
            code = line.split("//")[0]
            assert not re.search(r"\bhipMemset(D8|D16|D32|2D|3D)?\(", code), f"{os.path.basename(f)}:{k}: {line.strip()}"


def test_launches_name_a_stream():
    """Four arguments between <<< and >>>, the last one not zero."""
    for f in sorted(glob.glob(os.path.join(CSRC, "*.h*p"))):
        text = re.sub(r"//[^\n]*", "", open(f).read())
        for m in re.finditer(r"<<<(.*?)>>>", text, flags=re.S):
            cfg, depth, args = m.group(1), 0, 1
            for ch in cfg:
                depth += ch in "([{"
                depth -= ch in ")]}"
                args += ch == "," and depth == 0
            last = re.split(r",", cfg)[-1].strip(" \\\n")
            assert args == 4 and last not in ("0", "nullptr"), (os.path.basename(f), cfg)
