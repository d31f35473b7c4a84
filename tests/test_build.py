"""Every HIP source is what the language version of its build allows and compiles without a warning
(syntax only: no code is generated, no GPU needed)."""
import os
import subprocess

import pytest

from paper_2509_18824_amd import build as B


@pytest.mark.parametrize("source", B.sources())
def test_source_compiles_without_a_warning(source):
    # the host pass does not know the packed-fp32 feature and says so without a warning's name
    r = subprocess.run([B.HIPCC, *B.FLAGS, *B.FILE_FLAGS.get(source, []), "-Wno-unused-command-line-argument", "-fsyntax-only",
                        os.path.join(B.CSRC, source)], capture_output=True, text=True)
    lines = [l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l]
    assert r.returncode == 0 and not lines, "\n".join(lines)
