"""PPF_Q_WORKSPACE_BYTES counts every buffer the plan keeps per HIP stream: the
two-pass workspace and the partial sums of detection in parts."""
import pytest

from tests import launches

MIB = 1 << 20


@pytest.mark.parametrize("command,mib", [
    ("query 1024 8 0 0 64 0", 0),             # one launch, no buffer
    ("query 1024 8 0 0 4096 8", 0),           # detection in whole groups
    ("query 1024 8 0 0 64 64", 2),            # in parts, fused: 2 MiB of sums
    ("query 4096 8 0 0 64 64", 4),
    ("query 4096 32 0 0 64 0", 128),          # two passes
    ("query 4096 32 0 0 64 64", 128),         # in parts, two passes: in the workspace
])
def test_bytes(command, mib):
    (got,), = launches.run(command)
    assert int(got) == mib * MIB
