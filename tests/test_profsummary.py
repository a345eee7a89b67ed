"""The table that ties profile summaries to the kernels' sources: every kernel of the
library is in it with the file that defines it, and the hash a summary records covers
that file and every header a kernel's body may stand in."""
import glob
import os
import re
import shutil

import pytest

from paper_2205_13824_amd import profsummary as S

CSRC = os.path.join(S.HERE, "csrc")


def _kernels():
    out = {}
    for path in glob.glob(os.path.join(CSRC, "*.hip")):
        with open(path) as f:
            text = re.sub(r"//[^\n]*", "", f.read())
        for m in re.finditer(r"__global__[^;{]*?\b(k_\w+)\s*\(", text):
            out[m.group(1)] = os.path.basename(path)
    return out


def test_every_kernel_is_in_the_table():
    assert S.KERNEL_FILES == _kernels()


@pytest.mark.parametrize("changed", sorted(os.path.basename(p) for p in glob.glob(os.path.join(CSRC, "*.h"))))
def test_the_hash_covers_every_header(tmp_path, monkeypatch, changed):
    shutil.copytree(CSRC, tmp_path / "csrc")
    monkeypatch.setattr(S, "HERE", str(tmp_path))
    before = {k: S.kernel_sha16(k) for k in S.KERNEL_FILES}
    with open(tmp_path / "csrc" / changed, "a") as f:
        f.write("// changed\n")
    for k, h in before.items():
        assert S.kernel_sha16(k) != h
