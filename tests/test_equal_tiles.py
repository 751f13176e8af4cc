"""When the fused kernels at N = 512 and 1024 cut a batch of several rounds into
equal tiles instead of full-length ones: FP32 spectra only while the last round
is at most 5/8 full after one full round, an eighth less after each further one;
FP16 and int8 input and detection up to 5/8 always. (The probe reports two
workgroups per CU, so a round is 131072 spectra at N = 1024, 524288 at N = 512.)
"""
import pytest

from tests import launches


def grid(op, n, in_type, m):
    words, = launches.run(f"grid {op} {n} 8 {in_type} 0 {m} 16")
    name, workgroups = words[0].split(":")
    assert len(words) == 1 and launches.kernel(name) == "ppf_fused_kernel"
    return int(workgroups)


@pytest.mark.parametrize("n", [512, 1024])
@pytest.mark.parametrize("op,in_type", [("exec", 0), ("exec", 1), ("exec", 2), ("power", 0)])
@pytest.mark.parametrize("rounds", [1, 2, 3, 4, 5, 6, 7])
def test_rule(n, op, in_type, rounds):
    full = (2 << 20) // (8 * n)                       # spectra of a full-length tile
    groups = 1024 // n                                # tiles of a workgroup
    slots = 512 * groups
    most = 5 if op == "power" or in_type else 6 - rounds
    for eighths in (1, 2, 3, 4, 5, 6):
        for extra in (0, 1):                          # tiles beyond that many eighths
            tiles = slots * rounds + slots * eighths // 8 + extra
            got = grid(op, n, in_type, tiles * full)
            if eighths < most or (eighths == most and extra == 0):
                # detection's tiles are whole groups of 16 spectra: full-length ones at the most
                assert tiles - (op == "power") < got * groups <= slots * (rounds + 1), (eighths, extra, got)
            else:
                assert got == -(-tiles // groups), (eighths, extra, got)


def test_no_tiles_of_192_spectra():
    assert grid("exec", 1024, 0, 131072 * 3 // 2) == -(-131072 * 3 // 2 // 196)
