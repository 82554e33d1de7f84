"""Rules of the device code that are plain arithmetic, compiled for the host and run on the CPU: where
the tiles of an attention's part lie, up to the largest cache; the bounds on a table's
norms; the means' division."""
import os
import subprocess

import pytest

from paper_2602_02958_amd import build as qbuild

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_rules") / "host_rules")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *qbuild.FLAGS, "--offload-host-only", os.path.join(HERE, "host_rules.cpp"), "-o", exe],
                   check=True, stderr=subprocess.DEVNULL)
    text = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return dict(line.split(" ", 1) for line in text.splitlines())


@pytest.mark.parametrize("name", ["quotients", "norm_bounds", "norm_reaches", "tiles_small", "tiles_one_chunk", "tiles_top", "tiles_top_one_chunk", "tiles_top_undivided"])
def test_host_rule(rules, name):
    assert rules[name] == "ok"
