"""Which detection calls are cut into parts where halving a group saves little: a
half that gives CUs a second workgroup has to save two steps of four spectra
up to N = 1024, the tiles of a cut call
are single parts, and N = 128 has half the places.
"""
import pytest

from tests import launches


@pytest.mark.parametrize("n,taps,k_int,groups,cut,workgroups", [
    (1024, 8, 8, 64, 8, 128), (1024, 8, 8, 128, 4, 256),    # parts of one and two spectra share a step
    (1024, 8, 10, 256, 1, 256), (1024, 8, 12, 256, 1, 256), (1024, 8, 14, 256, 2, 512), (1024, 8, 16, 256, 2, 512),
    (1024, 8, 14, 171, 2, 342), (1024, 8, 10, 128, 2, 256), (1024, 8, 10, 64, 5, 160),
    (512, 8, 16, 512, 2, 512), (256, 8, 20, 1024, 2, 512), (256, 8, 16, 1024, 1, 256),
    (128, 8, 24, 2048, 1, 256), (128, 8, 32, 1025, 1, 129), (128, 8, 32, 1024, 2, 256), (2048, 8, 6, 128, 2, 256), (1024, 8, 10, 129, 1, 129),
])
def test_cut(n, taps, k_int, groups, cut, workgroups):
    words, = launches.run(f"grid power {n} {taps} 0 0 {k_int * groups} {k_int}")
    names = [w.rsplit(":", 1) for w in words]
    assert [launches.kernel(w) for w, _ in names] == ["ppf_fused_kernel"] + ["ppf_power_parts_kernel"] * (cut > 1)
    assert int(names[0][1]) == workgroups
    if cut > 1:
        assert int(names[1][1]) == groups
