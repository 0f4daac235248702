"""The traversals read one node layout (four children, quantized boxes).  Builds that
ask for another one, as options of earlier versions did, stop with an error instead of
giving a library whose rays read nodes of another size."""
import os
import shutil
import subprocess

import pytest

from paper_1903_07145_amd import build

HIPCC = os.environ.get("HIPCC", "hipcc")


def _compile(source, define):
    cmd = [HIPCC] + build.FLAGS + ["--cuda-host-only", "-fsyntax-only", os.path.join(build.CSRC, source)]
    return subprocess.run(cmd + (["-D" + define] if define else []), capture_output=True, text=True, timeout=300)


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not available")
@pytest.mark.parametrize("define,accepted", [(None, True), ("IPT_NODE_WIDTH=4", True), ("IPT_NODE_WIDTH=2", False),
                                             ("IPT_NODE_QUANT=0", False)])
def test_node_layout_is_no_option(define, accepted):
    r = _compile("stream.hip", define)
    if accepted:
        assert r.returncode == 0, r.stderr
    else:
        assert r.returncode != 0 and "node layout is fixed" in r.stderr
