"""Chunks of a two-pass call longer than the workspace (16384 spectra at N = 1024): equal
for FP32 input up to 32 taps, full ones and a rest otherwise."""
import pytest

from tests import launches


@pytest.mark.parametrize("taps,in_type,equal", [(32, 0, True), (33, 0, False), (40, 0, False), (64, 0, False),
                                                (32, 1, False), (40, 2, False)])
def test_chunks(taps, in_type, equal):
    words, = launches.run(f"grid exec 1024 {taps} {in_type} 2 34064")
    fft = [int(w.rsplit(":", 1)[1]) for w in words[1::2]]          # the FFT pass, workgroups by chunk
    assert len(fft) == 3 and fft[0] == fft[1]
    assert (fft[2] == fft[0]) == equal
