"""Tiles of batches with 2 taps: one spectrum each while every CU (256) has at most one
workgroup, two beyond that; with 4 taps one spectrum while there are free slots."""
import pytest

from tests import launches


@pytest.mark.parametrize("n,taps,in_type,m,workgroups", [
    (1024, 2, 0, 256, 256), (1024, 2, 0, 257, 129), (1024, 2, 1, 512, 256), (2048, 2, 2, 256, 256),
    (2048, 2, 0, 300, 150), (512, 2, 0, 512, 256), (512, 2, 0, 513, 129), (4096, 2, 0, 256, 256), (4096, 2, 0, 400, 200),
    (2048, 3, 0, 300, 300),
])
def test_workgroups(n, taps, in_type, m, workgroups):
    words, = launches.run(f"grid exec {n} {taps} {in_type} 0 {m}")
    assert int(words[0].split(":")[1]) == workgroups
